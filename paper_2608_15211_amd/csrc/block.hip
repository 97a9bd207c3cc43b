// block.hip - the rest of one Swin block around the window attention
// (Sec. IV-A Swin blocks; Sec. IV-C: the linear layers that TP shards;
// Table III model widths): LayerNorm, the QKV projection, the output
// projection and the GELU MLP, forward and backward, bf16 storage with
// float32 accumulation.
//
// One matrix-core GEMM kernel serves every linear layer.  Operands are
// bf16 row-major matrices in HBM, brought into XOR-swizzled LDS tiles by
// direct-to-LDS loads through a ring of stages; the 32 x 16 matrix-core
// operands are read either straight (when the contraction index runs along
// memory rows) or through the LDS transpose read (when it runs down memory
// columns), so Y = X W^T, dX = dY W and dW = dY^T X all take the same
// kernel.  In the forward each LayerNorm is folded into the projection
// after it (gains into the weights, mean and 1/std applied to the
// accumulators), so normalised activations never reach HBM there; the
// backward recomputes them once per weight gradient.  Bias, residual,
// GELU and its derivative are applied in the epilogue.
#include <algorithm>
#include <type_traits>

#include "terra_common.h"
#include "terra_block.h"

namespace terra {

typedef __bf16 bf16;
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s lds_v4s;

constexpr int kBM = 256;          // rows and columns of a workgroup tile, eight-wave form
constexpr int kBS = 128;          // four-wave form
constexpr int kBK = 64;           // contraction depth per stage
constexpr int kEpiS = 68;         // row stride (floats) of a wave's epilogue staging tile
constexpr int kMaxWgradSlices = 64;   // most token slices of a weight gradient
constexpr int kMaxCusBlock = 256;  // compute units the weight-gradient slices are sized for

// A bf16 operand in memory: row-major, `ld` elements a row, `rows` valid rows.
struct Mat {
  const bf16* p;
  int ld;
  int rows;
  // Three-part operand (read only by SEG kernels): three [rows][segw]
  // matrices side by side, part i at element offset i * segstride from p.
  int segw;
  int64_t segstride;
  __device__ const bf16* at(int r, int c) const { return p + (int64_t)r * ld + c; }
};


enum Epi {
  EPI_LN_QKV = 0,      // LayerNorm folded: out = bf16(rstd (acc - mean s) + c)   (column-split output)
  EPI_BIAS_RES = 1,    // out = bf16(acc + bias + res)
  EPI_LN_GELU = 2,     // t = rstd (acc - mean s) + c:  out = bf16(t), out2 = bf16(GELU(t))
  EPI_GELU_GRAD = 3,   // out = bf16(acc * GELU'(aux))
  EPI_F32 = 4,         // outf = acc (float32), slice blockIdx.z
  EPI_BF16 = 5,        // out = bf16(acc)
  EPI_F32_ACC = 6,     // outf += acc (float32)
};

struct EpiArgs {
  bf16* out[3];        // column-split bf16 output (split columns each)
  int split;
  bf16* out2;          // second bf16 output (GELU), ld = N
  const bf16* aux;     // residual or pre-activation, ld = N
  const float* bias;
  float* outf;         // float32 output, ld = N, slice stride M * N
  const float* mean;   // LayerNorm folded into the epilogue: per-row mean and 1/std,
  const float* rstd;   // per-column sum of the folded weights (lns) and constant (lnc)
  const float* lns;
  const float* lnc;
  // EPI_GELU_GRAD: column sums of the bf16 output over the rows of each wave
  // (half a tile's: 128, in the four-wave form 64), partial row 2 (tile row) +
  // (wave row), ld = N (nullable)
  float* colpart;
};

// Phi(x), the standard normal distribution function: with a = |x|,
// Phi(-a) = 2^P(a), P a degree-8 polynomial fitted to log2 Phi(-a) on
// [0, 5.6] (weighted minimax; P falls without bound beyond, where Phi(-a) <
// 1.1e-8).  Largest error as the hardware computes it, over 5e6 points from
// -40 to 40: Phi 5.7e-8 below zero and 8.2e-8 above (one minus it), GELU
// 4.0e-7, its derivative 1.3e-7.  One exponential and no division: the MLP
// epilogues are bound by vector instructions.  Against Abramowitz and
// Stegun's 7.1.26 (a reciprocal and an exponential: 2.9e-7, 4.7e-7 and 3.2e-7
// on the same points, and no interval where it is closer) the fc1 epilogue
// goes from 21.6 to 17.6 instructions an element and the 128 x 1080 fc1
// product from 1026 to 959 us, dh from 890 to 851.
__device__ inline float phi_f(float x) {
  const float a = fabsf(x);
  float p = -2.772049e-06f;
  p = fmaf(p, a, 3.8620746e-05f);
  p = fmaf(p, a, -1.8254759e-04f);
  p = fmaf(p, a, -1.4587014e-04f);
  p = fmaf(p, a, 7.0754718e-03f);
  p = fmaf(p, a, -5.2505028e-02f);
  p = fmaf(p, a, -0.45920491f);
  p = fmaf(p, a, -1.1511058f);
  p = fmaf(p, a, -1.0f);
  const float w = __builtin_amdgcn_exp2f(p);
  return x > 0.0f ? 1.0f - w : w;
}
__device__ inline float gelu_f(float x) { return x * phi_f(x); }
// Phi(x) + x phi(x), phi(x) = 2^(-x^2 log2(e) / 2 - log2(sqrt(2 pi)))
__device__ inline float gelu_grad_f(float x) {
  return fmaf(x, __builtin_amdgcn_exp2f(fmaf(x * x, -0.72134752f, -1.3257481f)), phi_f(x));
}

// ---------------------------------------------------------------------------
// LDS tiles.  A stage holds the A tile (kBM output rows x kBK) and the B tile
// (kBN x kBK), each in its memory layout, unpadded, with the 16-byte chunks
// of each row permuted by an XOR of the row index so that the matrix-core
// operand reads hit distinct banks:
// * KROW tile (memory [R][BK], BK / 8 chunks a row): chunk c of row r sits at
//   chunk c ^ ((r >> 1) & 7) - 16 consecutive rows read at one logical chunk
//   cover all 64 banks;
// * COLK tile (memory [BK][R], R / 8 chunks a row): chunk c of row k sits
//   at chunk c ^ (4 (k & 3)) - each half-wave of a transpose read takes 64
//   bytes from each of four rows, and these land on four different 64-byte
//   spans of the 256 bytes the LDS banks cover (measured: no bank conflicts;
//   with c ^ (2 (k & 3)) 0.8-2 conflict cycles per LDS instruction, though
//   no slower).
// ---------------------------------------------------------------------------
template <int R, bool KROW, int BK, int NT = 512>
struct Tile {
  static constexpr int kChunks = R * BK / 8;    // 16-byte chunks
  static constexpr int kPer = kChunks / NT;     // per thread (NT threads)
  static constexpr int kElems = R * BK;
  static constexpr int kCpr = BK / 8;           // chunks a row (KROW)
  __device__ static int swz(int row) { return (row >> 1) & 7; }
  // element offset of (row, logical chunk) of the memory layout
  __device__ static int off(int row, int c) {
    if (KROW) return row * BK + 8 * (c ^ swz(row));
    return row * R + 8 * (c ^ (4 * (row & 3)));
  }
  // memory (row, column) of the chunk stored in slot q (slot = chunk position in LDS order)
  __device__ static void slot_src(int q, int r0, int k0, int& mrow, int& mcol) {
    if (KROW) {
      const int row = q / kCpr, p = q % kCpr;
      mrow = r0 + row;
      mcol = k0 + 8 * (p ^ swz(row));
    } else {
      const int row = q / (R / 8), p = q - row * (R / 8);
      mrow = k0 + row;
      mcol = r0 + 8 * (p ^ (4 * (row & 3)));
    }
  }
};

// Straight operand (KROW tile): lane l receives T[m0 + l % 32][k0 + 8h + x],
// x = 0..7, h = l / 32, as one 16-byte read.
template <int R, int BK>
__device__ inline bf16x8 row_operand(const bf16* T, int k0, int m0, int lane) {
  const int row = m0 + (lane & 31);
  return *reinterpret_cast<const bf16x8*>(T + Tile<R, true, BK>::off(row, (k0 >> 3) + (lane >> 5)));
}

// Natural-order transposed operand (COLK tile): lane l receives
// T[k0 + 8h + x][m0 + l % 32], x = 0..7.  In each 16-lane group G of the
// transpose read, lane i gets element i % 4 of the 8 bytes that lane
// 16G + 4x + i/4 addresses, so lane L addresses row k0 + 8h + (L % 16) / 4
// (4 rows further for the second read), columns m0 + 16 (G % 2) + 4 (L % 4).
template <int R, int BK>
__device__ inline bf16x8 tr_operand(const bf16* T, int k0, int m0, int lane) {
  const int G = lane >> 4;
  const int row = k0 + 8 * (G >> 1) + ((lane & 15) >> 2);
  const int m = m0 + 16 * (G & 1) + 4 * (lane & 3);
  const int c = m >> 3, e = m & 7;
  const bf16* p0 = T + Tile<R, false, BK>::off(row, c) + e;
  const bf16* p1 = T + Tile<R, false, BK>::off(row + 4, c) + e;
  const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)p0);
  const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)p1);
  typedef short v8s __attribute__((ext_vector_type(8)));
  const v8s o = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, o);
}

// Direct-to-LDS staging of one operand tile: each thread moves kPer 16-byte
// chunks with buffer loads that write LDS themselves (slot q of the tile is
// written by thread q % NT, load q / NT); chunks outside the operand or the
// contraction slice read zeros.  The per-thread part of each chunk's address
// does not change along the contraction, so it is worked out once (init) and
// a stage costs one add and one bounds select a load.  KROW: the contraction
// index runs along memory rows.
template <int R, bool KROW, int BK, int NT>
struct Stager {
  typedef Tile<R, KROW, BK, NT> T;
  int voff[T::kPer];   // byte offset at contraction index 0 (2^31: outside the operand)
  int kpos[T::kPer];   // the chunk's contraction index inside a stage
  __device__ void init(const Mat& X, int r0, int nouter, int64_t base) {
#pragma unroll
    for (int u = 0; u < T::kPer; ++u) {
      int mr, mc;
      T::slot_src(u * NT + threadIdx.x, r0, 0, mr, mc);
      kpos[u] = KROW ? mc : mr;
      const bool ok = (KROW ? mr : mc) < nouter;
      voff[u] = ok ? (int)((base + (int64_t)mr * X.ld + mc) * 2) : (int)0x80000000;
    }
  }
  // koff: byte offset of the stage's first contraction index; krem:
  // contraction indices left from there
  __device__ void load(const i32x4& rs, bf16* tile, int koff, int krem) const {
    static_assert(T::kPer == 4, "one group of four loads");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: the LDS base goes to M0
    int v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = kpos[u] < krem ? voff[u] + koff : (int)0x80000000;
    buffer_load_lds16x4<16 * NT>(rs, tile + 8 * wave * 64, v);   // wave-uniform bases of 64 slots
  }
};


// C[M][N] = A[M][K] B[K][N] (+ epilogue).  AKROW: A is memory [M][K]
// (else [K][M]); BKROW: B is memory [N][K] (else [K][N]).  The grid holds
// (contraction slice, tile) pairs, slice z over [z * kslice, (z+1) * kslice).
// Eight waves, each a 128 x 64 block of the 256 x 256 tile.  SEG: A is a
// three-part operand split along K (AKROW; A.segw a multiple of kBK) or
// along M (else; A.segw a multiple of kBM), so that every stage (AKROW) or
// every workgroup tile (else) reads one part.
//
// What bounds it: the matrix cores and the L2 -> LDS stream about equally.
// On 131072 x 768 x 3072 the matrix instructions alone take 367 us (the
// clock drops to 1.9 GHz under them), the loads alone 361 us (4.8 GB through
// the L2s), the LDS reads hide under either; together 500 us, 1240 TFLOP/s.
// * The two waves of a SIMD (w and w + 4) take turns: while one half of the
//   workgroup issues its 32-deep matrix cluster, the other reads its next
//   operands from LDS and issues its loads, with a barrier after each turn.
//   Against all eight waves reading and then multiplying together: the same
//   product 620 -> 569 us, the weight gradients (transpose reads) 918 -> 603.
// * Stages are 64 deep, so that a K-major row piece is a whole 128-byte
//   line: the L2 serves half as many requests (569 -> 500 us).  Three stages
//   of A (activations, further away) and two of B fill the 160 KB of LDS.
// * Each XCD takes one contiguous run of (slice, tile) pairs whatever their
//   number, so that the tiles of one token slice share an L2 (weight
//   gradient of 3072 x 768: L2 misses 2.8e7 -> 1.1e7).
// NW = 4: four waves, each a 64 x 64 block of a 128 x 128 tile, for products
// whose 256 x 256 tiles would leave most CUs idle.  There the time is a
// workgroup's own chain of stages, so four stages of both operands keep
// three in flight (0.65 us a stage against 1.35 in the eight-wave form).
template <bool AKROW, bool BKROW, int EPI, bool SEG = false, int NW = 8>
__global__ __launch_bounds__(NW * 64, 1) void gemm_kernel(Mat A, Mat B, EpiArgs ep, int M, int N, int K,
                                                          int kslice) {
  constexpr int NT = NW * 64, BM = NW == 8 ? kBM : kBS, BN = BM, BK = kBK;
  constexpr int MI = BM / 64, kWM = 32 * MI;         // 32-row blocks and rows of a wave
  typedef Tile<BM, AKROW, BK, NT> TA;
  typedef Tile<BN, BKROW, BK, NT> TB;
  extern __shared__ __align__(16) char smem[];
  bf16* lds = reinterpret_cast<bf16*>(smem);

  const int nN = (N + BN - 1) / BN;
  const int nM = (M + BM - 1) / BM;
  const int tiles = nM * nN;
  // Workgroups go to the 8 XCDs in turn; each XCD takes one contiguous run
  // of (slice, tile) pairs, so that the tiles sharing operand rows sit
  // behind one L2.
  const int total = gridDim.x, xcd = blockIdx.x & 7;
  const int w0 = xcd * (total >> 3) + min(xcd, total & 7) + (blockIdx.x >> 3);
  const int z = w0 / tiles, w = w0 - z * tiles;
  const int tm = w / nN, tn = w - (w / nN) * nN;
  const int m0 = tm * BM, n0 = tn * BN;
  const int kbeg = z * kslice;
  const int kend = min(K, kbeg + kslice);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wm = (wave / (NW / 2)) * kWM, wn = (wave % (NW / 2)) * 64;
  const i32x4 rsa = buffer_rsrc(A.p, (uint32_t)(((int64_t)A.rows * A.ld + (SEG ? 2 * A.segstride : 0)) * 2));
  const i32x4 rsb = buffer_rsrc(B.p, (uint32_t)((int64_t)B.rows * B.ld * 2));

  f32x16 acc[MI][2];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};

  Stager<BM, AKROW, BK, NT> sa;
  Stager<BN, BKROW, BK, NT> sb;
  int seg = 0;
  if constexpr (SEG && !AKROW) {
    seg = m0 / A.segw;
    sa.init(A, m0 - seg * A.segw, min(M - seg * A.segw, A.segw), seg * A.segstride);
  } else {
    sa.init(A, m0, M, 0);
  }
  sb.init(B, n0, N, 0);
  const int kba = AKROW ? 2 : 2 * A.ld, kbb = BKROW ? 2 : 2 * B.ld;   // bytes per contraction index
  // LDS rings: kRA stages of A, then two (four waves: four) of B
  constexpr int kRA = NW == 8 ? 3 : 4;
  auto a_tile = [&](int st) { return lds + st * TA::kElems; };
  auto b_tile = [&](int st) { return lds + kRA * TA::kElems + st * TB::kElems; };
  auto issue_a = [&](int s, int st) {
    const int k0 = kbeg + s * BK;
    if constexpr (SEG && AKROW) {
      // the stage's part of the operand: its offset replaces the column's
      const int sg = k0 / A.segw;
      const int ks = k0 - sg * A.segw;
      sa.load(rsa, a_tile(st), (int)((sg * A.segstride + ks) * 2), min(kend - k0, A.segw - ks));
    } else {
      sa.load(rsa, a_tile(st), k0 * kba, kend - k0);
    }
  };
  auto issue_b = [&](int s, int st) {
    const int k0 = kbeg + s * BK;
    sb.load(rsb, b_tile(st), k0 * kbb, kend - k0);
  };

  const int nk = (kend - kbeg + BK - 1) / BK;
  bf16x8 ao[2][MI], bo[2][2];
  // operands of the 32 contraction indices from 32 * hf of a stage
  auto read_ops = [&](const bf16* ta, const bf16* tb, int hf) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int k0 = 32 * hf + 16 * c;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        bo[c][j] = BKROW ? row_operand<BN, BK>(tb, k0, wn + 32 * j, lane) : tr_operand<BN, BK>(tb, k0, wn + 32 * j, lane);
#pragma unroll
      for (int i = 0; i < MI; ++i)
        ao[c][i] =
            AKROW ? row_operand<BM, BK>(ta, k0, wm + 32 * i, lane) : tr_operand<BM, BK>(ta, k0, wm + 32 * i, lane);
    }
  };
  auto mfmas = [&]() {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) mma16(acc[i][j], ao[c][i], bo[c][j]);
  };
  if constexpr (NW == 8) {
    // Turn 4 kt + 2 hf: the first half of the workgroup reads half hf of
    // stage kt, the second half multiplies what it read in its last turn;
    // in the next turn they swap.  A stage's buffer is free after turn
    // 4 kt + 3, so the loads of B's stage kt + 1 (two buffers) go out while
    // half 0 of stage kt is read, those of A's stage kt + 2 (three) while
    // half 1 is.
    const bool second = __builtin_amdgcn_readfirstlane(wave) >= NW / 2;
    if (nk > 0) {
      issue_a(0, 0);
      issue_b(0, 0);
    }
    if (nk > 1) {
      issue_a(1, 1);
      wait_vm<TA::kPer>();
    } else {
      wait_vm<0>();
    }
    lds_barrier();
    if (second) lds_barrier();
    int sa3 = 0;               // kt % 3
    for (int kt = 0; kt < nk; ++kt) {
      const bf16* ta = a_tile(sa3);
      const bf16* tb = b_tile(kt & 1);
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        read_ops(ta, tb, hf);
        if (hf == 0) {
          if (kt + 1 < nk) issue_b(kt + 1, (kt + 1) & 1);
        } else {
          if (kt + 2 < nk) issue_a(kt + 2, sa3 == 0 ? 2 : sa3 - 1);
        }
        auto wait_next = [&]() {     // stage kt + 1 is in LDS (A of stage kt + 2 may be in flight)
          if (hf == 1) {
            if (kt + 2 < nk) wait_vm<TA::kPer>();
            else wait_vm<0>();
          }
        };
        if (second) wait_next();
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
        mfmas();
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        if (!second) wait_next();
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      sa3 = sa3 == 2 ? 0 : sa3 + 1;
    }
    if (!second) lds_barrier();
  } else {
    constexpr int kLoads = TA::kPer + TB::kPer;
    for (int s = 0; s < 3; ++s)
      if (s < nk) { issue_a(s, s); issue_b(s, s); }
    for (int kt = 0; kt < nk; ++kt) {
      const int left = nk - 1 - kt;      // stages after this one
      if (left >= 2) wait_vm<2 * kLoads>();
      else if (left == 1) wait_vm<kLoads>();
      else wait_vm<0>();
      lds_barrier();     // stage kt is in LDS, and every wave is done with the one before
      if (left >= 3) {
        issue_a(kt + 3, (kt + 3) & 3);
        issue_b(kt + 3, (kt + 3) & 3);
      }
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        read_ops(a_tile(kt & 3), b_tile(kt & 3), hf);
        mfmas();
      }
    }
  }
  __syncthreads();   // every wave is done with the stages: their LDS now stages the epilogue

  // Epilogue, 32 rows of the wave's block at a time: acc[i][j] holds rows
  // 32i + 8g + 4h + x (register 4g + x), column 32j + lane % 32; they go
  // through the wave's own LDS tile so that each lane then handles 8
  // consecutive columns of rows 8t + lane / 8, t = 0..3: eight lanes cover
  // the 64 columns of a row, so every 16-byte load or store instruction
  // moves whole 128-byte row pieces (bf16), and a lane keeps one set of 8
  // columns, whose constants it loads once.
  float* et = reinterpret_cast<float*>(smem) + wave * 32 * kEpiS;
  const int h = lane >> 5, col = lane & 31;
  const int er = lane >> 3, ec = (lane & 7) * 8;
  const int n = n0 + wn + ec;                          // N is a multiple of 8
  constexpr bool kCol = EPI == EPI_GELU_GRAD;
  float cs[8] = {};                                    // this lane's column sums over its rows
  // per-column epilogue constants (LayerNorm fold: s and c; bias)
  constexpr bool kLn = EPI == EPI_LN_QKV || EPI == EPI_LN_GELU;
  constexpr int kPc = kLn ? 2 : (EPI == EPI_BIAS_RES ? 1 : 0);
  float pc[2][8];
#pragma unroll
  for (int a = 0; a < kPc; ++a) {
    const float* src = kLn ? (a == 0 ? ep.lns : ep.lnc) : ep.bias;
    float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
    if (n < N) {
      lo = *reinterpret_cast<const float4*>(src + n);
      hi = *reinterpret_cast<const float4*>(src + n + 4);
    }
    pc[a][0] = lo.x; pc[a][1] = lo.y; pc[a][2] = lo.z; pc[a][3] = lo.w;
    pc[a][4] = hi.x; pc[a][5] = hi.y; pc[a][6] = hi.z; pc[a][7] = hi.w;
  }
  // Row inputs of one 32-row block (residual or pre-activation pieces, or
  // the rows' mean and 1/std), fetched one block ahead.  Tiles inside the
  // matrix take a form without bounds checks: no branch then separates the
  // loads, which all go out together.
  constexpr bool kAux = EPI == EPI_BIAS_RES || EPI == EPI_GELU_GRAD;
  struct RowIn {
    bf16x8 aux[kAux ? 4 : 1];
    float mu[kLn ? 4 : 1], rs[kLn ? 4 : 1];
  };
  auto epilogue = [&](auto full_c) {
    constexpr bool kFull = decltype(full_c)::value;
    auto inside = [&](int m) { return kFull || (m < M && n < N); };
    auto fetch = [&](int i, RowIn& in) {
#pragma unroll
      for (int t4 = 0; t4 < 4; ++t4) {
        const int m = m0 + wm + 32 * i + 8 * t4 + er;
        if (kAux) {
          in.aux[t4] = bf16x8{};
          if (inside(m)) in.aux[t4] = *reinterpret_cast<const bf16x8*>(ep.aux + (int64_t)m * N + n);
        }
        if (kLn) {
          in.mu[t4] = inside(m) ? ep.mean[m] : 0.0f;
          in.rs[t4] = inside(m) ? ep.rstd[m] : 0.0f;
        }
      }
    };
    RowIn in[2];
    if (kAux || kLn) fetch(0, in[0]);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) et[(8 * (r / 4) + 4 * h + (r % 4)) * kEpiS + 32 * j + col] = acc[i][j][r];
      if ((kAux || kLn) && i < MI - 1) fetch(i + 1, in[(i + 1) & 1]);
      __builtin_amdgcn_wave_barrier();
      const RowIn& ri = in[i & 1];
#pragma unroll
      for (int t4 = 0; t4 < 4; ++t4) {
        const int m = m0 + wm + 32 * i + 8 * t4 + er;
        const float4 lo = *reinterpret_cast<const float4*>(et + (8 * t4 + er) * kEpiS + ec);
        const float4 hi = *reinterpret_cast<const float4*>(et + (8 * t4 + er) * kEpiS + ec + 4);
        float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        const int64_t o = (int64_t)m * N + n;
        if (EPI == EPI_F32 || EPI == EPI_F32_ACC) {
          if (!inside(m)) continue;
          float* dst = ep.outf + (EPI == EPI_F32 ? (int64_t)z * M * N : 0) + o;
          if (EPI == EPI_F32_ACC) {
            const float4 a0 = *reinterpret_cast<const float4*>(dst);
            const float4 a1 = *reinterpret_cast<const float4*>(dst + 4);
            v[0] += a0.x; v[1] += a0.y; v[2] += a0.z; v[3] += a0.w;
            v[4] += a1.x; v[5] += a1.y; v[6] += a1.z; v[7] += a1.w;
          }
          *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
          *reinterpret_cast<float4*>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
          continue;
        }
        bf16x8 t, u;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          float y = v[x];
          if (kLn) y = ri.rs[t4] * (y - ri.mu[t4] * pc[0][x]) + pc[1][x];
          if (EPI == EPI_BIAS_RES) y = y + pc[0][x] + (float)ri.aux[t4][x];
          if (EPI == EPI_GELU_GRAD) y *= gelu_grad_f((float)ri.aux[t4][x]);
          t[x] = (bf16)y;
          if (EPI == EPI_LN_GELU) u[x] = (bf16)gelu_f(y);
        }
        if (!inside(m)) continue;
        if (EPI == EPI_LN_QKV) {
          const int blk = n / ep.split;
          *reinterpret_cast<bf16x8*>(ep.out[blk] + (int64_t)m * ep.split + (n - blk * ep.split)) = t;
        } else {
          *reinterpret_cast<bf16x8*>(ep.out[0] + o) = t;
        }
        if (EPI == EPI_LN_GELU) *reinterpret_cast<bf16x8*>(ep.out2 + o) = u;
        if (kCol) {
#pragma unroll
          for (int x = 0; x < 8; ++x) cs[x] += (float)t[x];
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  };
  if (m0 + BM <= M && n0 + BN <= N) epilogue(std::true_type{});
  else epilogue(std::false_type{});
  if constexpr (kCol) {
    // lanes 8t + c (t = 0..7) hold 16-row sums of columns 8c..8c+7: through
    // the wave's staging tile, lane l then adds column l over them in order
    if (ep.colpart != nullptr) {
#pragma unroll
      for (int x = 0; x < 8; ++x) et[er * kEpiS + ec + x] = cs[x];
      __builtin_amdgcn_wave_barrier();
      float sum = 0.0f;
#pragma unroll
      for (int r = 0; r < 8; ++r) sum += et[r * kEpiS + lane];
      if (n0 + wn + lane < N) ep.colpart[(int64_t)(2 * tm + wm / kWM) * N + n0 + wn + lane] = sum;
    }
  }
}

// LayerNorm applied to a token matrix (the backward's weight gradients take
// the normalised activations as an operand): out = (z - mean) rstd gamma +
// beta, rounded to bf16; one thread per 8 channels.
__device__ inline void ln_apply_rows(int block, const bf16* __restrict__ z, const float* __restrict__ mean,
                                     const float* __restrict__ rstd, const float* __restrict__ gamma,
                                     const float* __restrict__ beta, bf16* __restrict__ out, int T, int C) {
  const int64_t idx = (int64_t)block * 256 + threadIdx.x;
  const int c8 = C / 8;
  if (idx >= (int64_t)T * c8) return;
  const int t = (int)(idx / c8);
  const int c = 8 * (int)(idx - (int64_t)t * c8);
  const bf16x8 v = *reinterpret_cast<const bf16x8*>(z + (int64_t)t * C + c);
  const float mu = mean[t], rs = rstd[t];
  bf16x8 o;
#pragma unroll
  for (int x = 0; x < 8; ++x) o[x] = (bf16)(((float)v[x] - mu) * rs * gamma[c + x] + beta[c + x]);
  *reinterpret_cast<bf16x8*>(out + (int64_t)t * C + c) = o;
}
__global__ __launch_bounds__(256) void ln_apply_kernel(const bf16* __restrict__ z, const float* __restrict__ mean,
                                                      const float* __restrict__ rstd, const float* __restrict__ gamma,
                                                      const float* __restrict__ beta, bf16* __restrict__ out, int T,
                                                      int C) {
  ln_apply_rows(blockIdx.x, z, mean, rstd, gamma, beta, out, T, C);
}

// LayerNorm folded into the following linear layer: with
// LN(x)_k = (x_k - mean) rstd gamma_k + beta_k,
//   LN(x) W^T + b = rstd (x Wf^T - mean s) + c,
//   Wf[n][k] = bf16(W[n][k] gamma_k),  s_n = sum_k Wf[n][k],
//   c_n = b_n + sum_k W[n][k] beta_k,
// so the GEMM runs on the raw activations and the epilogue normalises.  One
// wave per output row n.
__device__ inline void ln_fold(int block, const bf16* __restrict__ W, const float* __restrict__ gamma,
                               const float* __restrict__ beta, const float* __restrict__ bias,
                               bf16* __restrict__ Wf, float* __restrict__ lns,
                               float* __restrict__ lnc, int N, int K) {
  const int n = block * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (n >= N) return;
  float sacc = 0.0f, cacc = 0.0f;
  for (int k = 8 * lane; k < K; k += 512) {
    const bf16x8 w = *reinterpret_cast<const bf16x8*>(W + (int64_t)n * K + k);
    bf16x8 f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      f[i] = (bf16)((float)w[i] * gamma[k + i]);
      sacc += (float)f[i];
      cacc += (float)w[i] * beta[k + i];
    }
    *reinterpret_cast<bf16x8*>(Wf + (int64_t)n * K + k) = f;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    sacc += __shfl_xor(sacc, o, 64);
    cacc += __shfl_xor(cacc, o, 64);
  }
  if (lane == 0) {
    lns[n] = sacc;
    lnc[n] = cacc + bias[n];
  }
}

// ---------------------------------------------------------------------------
// LayerNorm statistics: one wave per token, mean and 1 / sqrt(var + eps)
// (biased variance, two passes over the row).
// ---------------------------------------------------------------------------
constexpr int kRowThreads = 256;

__device__ inline float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Mean and 1/std of each row, one wave a row: the row is read once into
// registers (C <= 2048: four 8-element chunks a lane) and the variance is
// taken about the mean from there.
__device__ inline void ln_stats_rows(int block, const bf16* __restrict__ x, float* __restrict__ mean,
                                     float* __restrict__ rstd, int T, int C, float eps) {
  const int row = block * (kRowThreads / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= T) return;
  const bf16* p = x + (int64_t)row * C;
  bf16x8 v[4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (8 * lane + 512 * c < C) v[c] = *reinterpret_cast<const bf16x8*>(p + 8 * lane + 512 * c);
  float s = 0.0f;
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (8 * lane + 512 * c < C)
#pragma unroll
      for (int i = 0; i < 8; ++i) s += (float)v[c][i];
  const float mu = wave_sum(s) / (float)C;
  float q = 0.0f;
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (8 * lane + 512 * c < C)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float d = (float)v[c][i] - mu;
        q += d * d;
      }
  const float var = wave_sum(q) / (float)C;
  if (lane == 0) {
    mean[row] = mu;
    rstd[row] = 1.0f / sqrtf(var + eps);
  }
}

__global__ __launch_bounds__(kRowThreads) void ln_stats_kernel(const bf16* __restrict__ x, float* __restrict__ mean,
                                                               float* __restrict__ rstd, int T, int C, float eps) {
  ln_stats_rows(blockIdx.x, x, mean, rstd, T, C, eps);
}

// One launch for what the forward needs before its products: the statistics
// of x (blocks [0, b0)) and the two folded weights (W_qkv in [b0, b1), W_fc1
// from b1).  Three launches of about 5 us each on small grids before.
struct FoldArgs {
  const bf16* W;
  const float *gamma, *beta, *bias;
  bf16* Wf;
  float *lns, *lnc;
  int N;
};
__global__ __launch_bounds__(kRowThreads) void block_prep_kernel(const bf16* __restrict__ x, float* __restrict__ mean,
                                                                 float* __restrict__ rstd, int T, int C, float eps,
                                                                 FoldArgs f0, FoldArgs f1, int b0, int b1) {
  const int b = blockIdx.x;
  if (b < b0) return ln_stats_rows(b, x, mean, rstd, T, C, eps);
  const FoldArgs& f = b < b1 ? f0 : f1;
  ln_fold(b - (b < b1 ? b0 : b1), f.W, f.gamma, f.beta, f.bias, f.Wf, f.lns, f.lnc, f.N, C);
}

// ---------------------------------------------------------------------------
// LayerNorm backward plus the residual branch, one wave per token:
//   g = dy * gamma, dz = rstd (g - mean(g) - zhat mean(g zhat)) + dres
// written as bf16; per-wave partial sums of dy * zhat (dgamma) and dy
// (dbeta) over the wave's tokens go to `part` ([wave][2][C]) for a
// fixed-order reduction.  Each lane owns channel chunks 8 (lane + 64 c).
// ---------------------------------------------------------------------------

// NCH = ceil(C / 512) chunk slots a lane (registers for C, not for 2048)
template <typename DY, int NCH>
__global__ __launch_bounds__(kRowThreads) void ln_bwd_kernel(
    const DY* __restrict__ dy, const bf16* __restrict__ z, const float* __restrict__ mean,
    const float* __restrict__ rstd, const float* __restrict__ gamma, const bf16* __restrict__ dres,
    bf16* __restrict__ dz, float* __restrict__ part, int T, int C, int rows_per_wave) {
  const int gw = blockIdx.x * (kRowThreads / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  float dg[NCH][8], db[NCH][8];
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int i = 0; i < 8; ++i) dg[c][i] = db[c][i] = 0.0f;
  const int r0 = gw * rows_per_wave;
  const int r1 = min(T, r0 + rows_per_wave);
  const float invC = 1.0f / (float)C;
  for (int row = r0; row < r1; ++row) {
    const float mu = mean[row], rs = rstd[row];
    float zh[NCH][8], gg[NCH][8];
    float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int ch = 8 * (lane + 64 * c);
      if (ch < C) {
        const bf16x8 zv = *reinterpret_cast<const bf16x8*>(z + (int64_t)row * C + ch);
        float d[8];
        if constexpr (sizeof(DY) == 4) {
          const float4 d0 = *reinterpret_cast<const float4*>(dy + (int64_t)row * C + ch);
          const float4 d1 = *reinterpret_cast<const float4*>(dy + (int64_t)row * C + ch + 4);
          d[0] = d0.x; d[1] = d0.y; d[2] = d0.z; d[3] = d0.w; d[4] = d1.x; d[5] = d1.y; d[6] = d1.z; d[7] = d1.w;
        } else {
          const bf16x8 dv = *reinterpret_cast<const bf16x8*>(dy + (int64_t)row * C + ch);
#pragma unroll
          for (int i = 0; i < 8; ++i) d[i] = (float)dv[i];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          zh[c][i] = ((float)zv[i] - mu) * rs;
          gg[c][i] = d[i] * gamma[ch + i];
          s1 += gg[c][i];
          s2 += gg[c][i] * zh[c][i];
          dg[c][i] += d[i] * zh[c][i];
          db[c][i] += d[i];
        }
      }
    }
    s1 = wave_sum(s1) * invC;
    s2 = wave_sum(s2) * invC;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int ch = 8 * (lane + 64 * c);
      if (ch < C) {
        const bf16x8 rv = *reinterpret_cast<const bf16x8*>(dres + (int64_t)row * C + ch);
        bf16x8 o;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = (bf16)(rs * (gg[c][i] - s1 - zh[c][i] * s2) + (float)rv[i]);
        *reinterpret_cast<bf16x8*>(dz + (int64_t)row * C + ch) = o;
      }
    }
  }
  float* pg = part + (int64_t)gw * 2 * C;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int ch = 8 * (lane + 64 * c);
    if (ch < C) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        pg[ch + i] = dg[c][i];
        pg[C + ch + i] = db[c][i];
      }
    }
  }
}

// Column sums of a bf16 matrix, per slice of rows:
// part[s][col] = sum over rows [s * rows_per, (s+1) * rows_per) - the bias
// gradients, reduced afterwards in slice order.  Thread = 8 columns.
__global__ __launch_bounds__(kRowThreads) void colsum_kernel(Mat X, int ncols, float* __restrict__ part,
                                                             int rows_per) {
  const int c8 = blockIdx.x * kRowThreads + threadIdx.x;
  if (8 * c8 >= ncols) return;
  const int s = blockIdx.y;
  const int r0 = s * rows_per, r1 = min(X.rows, r0 + rows_per);
  // a three-part X (segw > 0): column c of part c / segw
  const bf16* xb = X.p;
  int col = 8 * c8;
  if (X.segw > 0) {
    const int sg = col / X.segw;
    xb += sg * X.segstride;
    col -= sg * X.segw;
  }
  auto at = [&](int r) { return reinterpret_cast<const bf16x8*>(xb + (int64_t)r * X.ld + col); };
  // four independent partial sums (rows r, r+1, r+2, r+3 of each step), so
  // that four loads are in flight; combined in a fixed order at the end
  float acc[4][8] = {};
  int r = r0;
  for (; r + 4 <= r1; r += 4) {
    bf16x8 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = *at(r + u);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[u][i] += (float)v[u][i];
  }
  for (; r < r1; ++r) {
    const bf16x8 v = *at(r);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[0][i] += (float)v[i];
  }
#pragma unroll
  for (int i = 0; i < 8; ++i)
    part[(int64_t)s * ncols + 8 * c8 + i] = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
}

// The same in one launch, for up to kColDirect rows (a second launch costs
// more than the few workgroups' longer walk): a workgroup takes 64 columns
// (ncols is a multiple of 64, a part's width too), thread (r, c) the rows
// r, r + 32, ... of columns 8c .. 8c + 7; the 32 sums are added in order.
constexpr int kColDirect = 2048;
__global__ __launch_bounds__(256) void colsum_direct_kernel(Mat X, float* __restrict__ out) {
  __shared__ float red[32][65];
  const int c = threadIdx.x & 7, r0 = threadIdx.x >> 3;
  const bf16* xb = X.p;
  int col = 64 * blockIdx.x + 8 * c;
  if (X.segw > 0) {
    const int sg = col / X.segw;
    xb += sg * X.segstride;
    col -= sg * X.segw;
  }
  float acc[8] = {};
#pragma unroll 4
  for (int r = r0; r < X.rows; r += 32) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(xb + (int64_t)r * X.ld + col);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] += (float)v[i];
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) red[r0][8 * c + i] = acc[i];
  __syncthreads();
  if (threadIdx.x < 64) {
    float sum = 0.0f;
#pragma unroll
    for (int r = 0; r < 32; ++r) sum += red[r][threadIdx.x];
    out[64 * blockIdx.x + threadIdx.x] = sum;
  }
}

// grp[g][i] = sum of part[s][i] over s in [g * per, (g + 1) * per), in
// order (n entries per slice).
__global__ __launch_bounds__(kRowThreads) void group_sum_kernel(const float* __restrict__ part, float* __restrict__ grp,
                                                                int n, int per) {
  const int i = blockIdx.x * kRowThreads + threadIdx.x;
  if (i >= n) return;
  const int g = blockIdx.y;
  float acc = 0.0f;
  for (int sl = g * per; sl < (g + 1) * per; ++sl) acc += part[(int64_t)sl * n + i];
  grp[(int64_t)g * n + i] = acc;
}

// out[i] = sum over s < nslice of part[s * stride + i], in slice order (few
// slices, many outputs: the weight gradients).
__global__ __launch_bounds__(kRowThreads) void slice_sum_kernel(const float* __restrict__ part, float* __restrict__ out,
                                                                int64_t n, int64_t stride, int nslice) {
  const int64_t i = (int64_t)blockIdx.x * kRowThreads + threadIdx.x;
  if (i >= n) return;
  float acc = 0.0f;
  int s = 0;
  for (; s + 8 <= nslice; s += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(s + u) * stride + i];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  for (; s < nslice; ++s) acc += part[(int64_t)s * stride + i];
  out[i] = acc;
}

// The same for many slices and few outputs (the column sums' 512 row
// slices): a workgroup takes 64 consecutive i; its four waves sum the slices
// s = 4j + wave in order, and the four sums are added in wave order (a fixed
// order for every i), so that the slice list is four short dependent chains.
// Outputs from n0 on go to out1 (the LayerNorm shift beside the gain).
__global__ __launch_bounds__(256) void slice_sum4_kernel(const float* __restrict__ part, float* __restrict__ out,
                                                        float* __restrict__ out1, int64_t n0, int64_t n,
                                                        int64_t stride, int nslice) {
  __shared__ float red[4][64];
  const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + c;
  float acc = 0.0f;
  if (i < n) {
    int s = q;
    for (; s + 28 < nslice; s += 32) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(s + 4 * u) * stride + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; s < nslice; s += 4) acc += part[(int64_t)s * stride + i];
  }
  red[q][c] = acc;
  __syncthreads();
  if (q == 0 && i < n) (i < n0 ? out[i] : out1[i - n0]) = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
}

// out[c][r] = in[r][c] for a rows x cols bf16 matrix: the backward's copies
// of the weights in [N][K] order, so that its data-gradient products read
// their B operand with straight rather than transposed LDS reads (a few MB,
// once per backward).
__device__ inline void transpose_tile(int block, const bf16* __restrict__ in, bf16* __restrict__ out, int rows,
                                      int cols) {
  __shared__ bf16 t[32][33];
  const int nc = (cols + 31) / 32;
  const int c0 = (block % nc) * 32, r0 = (block / nc) * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int y = ty; y < 32; y += 8) {
    const int r = r0 + y, c = c0 + tx;
    if (r < rows && c < cols) t[y][tx] = in[(int64_t)r * cols + c];
  }
  __syncthreads();
  for (int y = ty; y < 32; y += 8) {
    const int c = c0 + y, r = r0 + tx;
    if (c < cols && r < rows) out[(int64_t)c * rows + r] = t[tx][y];
  }
}


// One launch for what the backward needs before its products: the four
// weight copies (blocks below b[3]) and LN2's output (from b[3]).  Five
// launches of about 5 us each on small grids before.
struct BwdPrep {
  const bf16* in[4];
  bf16* out[4];
  int rows[4], cols[4];
  int b[4];                // first block after each matrix
};
__global__ __launch_bounds__(256) void block_bwd_prep_kernel(BwdPrep w, const bf16* __restrict__ z,
                                                            const float* __restrict__ mean,
                                                            const float* __restrict__ rstd,
                                                            const float* __restrict__ gamma,
                                                            const float* __restrict__ beta, bf16* __restrict__ out,
                                                            int T, int C) {
  const int blk = blockIdx.x;
  if (blk >= w.b[3]) return ln_apply_rows(blk - w.b[3], z, mean, rstd, gamma, beta, out, T, C);
  int i = 0;
  while (blk >= w.b[i]) ++i;
  transpose_tile(blk - (i > 0 ? w.b[i - 1] : 0), w.in[i], w.out[i], w.rows[i], w.cols[i]);
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
// Contraction indices of each of ns slices: whole stages.
static int slice_len(int K, int ns) { return ((K + ns - 1) / ns + kBK - 1) / kBK * kBK; }

template <bool AKROW, bool BKROW, int EPI, bool SEG, int NW>
static hipError_t gemm_form(const Mat& A, const Mat& B, const EpiArgs& ep, int M, int N, int K, int nsplit,
                            hipStream_t st) {
  constexpr int BM = NW == 8 ? kBM : kBS;
  // stages of A and B: 3 + 2 of 32 KB (160 KB), or 4 + 4 of 16 KB (128 KB)
  constexpr size_t lds = (NW == 8 ? 5 : 8) * (size_t)BM * kBK * sizeof(bf16);
  const int tiles = ((M + BM - 1) / BM) * ((N + BM - 1) / BM);
  const int kslice = slice_len(K, nsplit);
  hipLaunchKernelGGL((gemm_kernel<AKROW, BKROW, EPI, SEG, NW>), dim3(tiles * nsplit), dim3(NW * 64), lds, st, A, B,
                     ep, M, N, K, kslice);
  return hipGetLastError();
}

// Which form a product takes, and in how many contraction slices (float32
// partials, summed in slice order).  Times in us from the kernels' own: a
// stage takes 1.35 in the eight-wave form and 0.65 in the four-wave one, a
// workgroup 8 and 3 besides (prologue, epilogue), a sum of slices 5 and its
// traffic; workgroups run in rounds of one per CU.
struct Plan {
  int nw, ns;
};
// The plan without slices past the contraction's end (2056 tokens in eight
// slices of 320 end in the seventh).
static Plan without_empty(Plan p, int K) {
  const int len = slice_len(K, p.ns);
  return {p.nw, (K + len - 1) / len};
}
static double plan_cost(int M, int N, int K, Plan p) {
  const int bm = p.nw == 8 ? kBM : kBS;
  const int tiles = ((M + bm - 1) / bm) * ((N + bm - 1) / bm);
  const int rounds = (tiles * p.ns + kMaxCusBlock - 1) / kMaxCusBlock;
  const int stages = ((K + p.ns - 1) / p.ns + kBK - 1) / kBK;
  const double sum = p.ns > 1 ? 5.0 + 2e-6 * p.ns * M * N : 0.0;
  return rounds * (p.nw == 8 ? 1.35 * stages + 8.0 : 0.65 * stages + 3.0) + sum;
}
static Plan plan_product(int M, int N, int K, int max_split) {
  Plan best = {8, 1};
  double c = plan_cost(M, N, K, best);
  for (int ns = 1; ns <= max_split && (ns == 1 || K >= 4 * kBK * ns); ++ns) {
    const double d = plan_cost(M, N, K, {4, ns});
    if (d < c) { c = d; best = {4, ns}; }
  }
  return without_empty(best, K);
}

template <bool AKROW, bool BKROW, int EPI, bool SEG = false>
static hipError_t gemm(const Mat& A, const Mat& B, const EpiArgs& ep, int M, int N, int K, hipStream_t st) {
  if (plan_product(M, N, K, 1).nw == 8) return gemm_form<AKROW, BKROW, EPI, SEG, 8>(A, B, ep, M, N, K, 1, st);
  return gemm_form<AKROW, BKROW, EPI, SEG, 4>(A, B, ep, M, N, K, 1, st);
}

// out = bf16(sum over slices of part [+ bias + res]), the end of a product
// in contraction slices; a thread takes 8 columns of one row.
template <int EPI>
__global__ __launch_bounds__(256) void split_sum_kernel(const float* __restrict__ part, EpiArgs ep, int64_t mn, int N,
                                                       int ns) {
  const int64_t o = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (o >= mn) return;
  float v[8] = {};
  for (int s = 0; s < ns; ++s) {
    const float4 lo = *reinterpret_cast<const float4*>(part + s * mn + o);
    const float4 hi = *reinterpret_cast<const float4*>(part + s * mn + o + 4);
    v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
    v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
  }
  bf16x8 t;
  if (EPI == EPI_BIAS_RES) {
    const float* b = ep.bias + o % N;
    const bf16x8 res = *reinterpret_cast<const bf16x8*>(ep.aux + o);
#pragma unroll
    for (int x = 0; x < 8; ++x) t[x] = (bf16)(v[x] + b[x] + (float)res[x]);
  } else {
#pragma unroll
    for (int x = 0; x < 8; ++x) t[x] = (bf16)v[x];
  }
  *reinterpret_cast<bf16x8*>(ep.out[0] + o) = t;
}

// Most slices of a product over K = 3C or 4C with few tiles, and the
// float32 partials they need.
constexpr int kMaxSplit = 8;
static size_t split_floats(int T, int C, int K) {
  const Plan p = plan_product(T, C, K, kMaxSplit);
  return p.ns > 1 ? (size_t)p.ns * T * C : 0;
}

static Mat mat(const void* p, int ld, int rows) {
  Mat m;
  m.p = (const bf16*)p;
  m.ld = ld;
  m.rows = rows;
  m.segw = 0;
  m.segstride = 0;
  return m;
}

// A long product with N = C (K-major A; bf16 or bias + residual epilogue):
// * few tiles: in contraction slices, finished by split_sum_kernel;
// * many: the rows of whole rounds of one 256 x 256 tile per CU, then the
//   rest (3 column tiles by ceil(T / 256) row tiles are 6.3 rounds on the
//   128x1080 grid at C = 768) as a product of its own.
template <bool BKROW, int EPI, bool SEG = false>
static hipError_t gemm_rounds(const Mat& A, const Mat& B, const EpiArgs& ep, int M, int N, int K, float* part,
                              hipStream_t st) {
  static_assert(EPI == EPI_BF16 || EPI == EPI_BIAS_RES, "row offsets are set for these epilogues");
  const Plan p = plan_product(M, N, K, kMaxSplit);
  if (p.ns > 1) {
    EpiArgs pe = {};
    pe.outf = part;
    const hipError_t e = gemm_form<true, BKROW, EPI_F32, SEG, 4>(A, B, pe, M, N, K, p.ns, st);
    if (e != hipSuccess) return e;
    const int64_t mn = (int64_t)M * N;
    hipLaunchKernelGGL((split_sum_kernel<EPI>), dim3((unsigned)((mn / 8 + 255) / 256)), dim3(256), 0, st, part, ep, mn,
                       N, p.ns);
    return hipGetLastError();
  }
  const int ntn = (N + kBM - 1) / kBM, nM = (M + kBM - 1) / kBM;
  const int r1 = ((nM * ntn) / kMaxCusBlock) * kMaxCusBlock / ntn;   // row tiles in whole rounds
  if (r1 == 0 || r1 >= nM) return gemm<true, BKROW, EPI, SEG>(A, B, ep, M, N, K, st);
  const int m1 = r1 * kBM;
  const hipError_t e = gemm_form<true, BKROW, EPI, SEG, 8>(A, B, ep, m1, N, K, 1, st);
  if (e != hipSuccess) return e;
  Mat a2 = A;
  a2.p = A.p + (int64_t)m1 * A.ld;
  a2.rows = A.rows - m1;
  EpiArgs e2 = ep;
  e2.out[0] = ep.out[0] + (int64_t)m1 * N;
  if (EPI == EPI_BIAS_RES) e2.aux = ep.aux + (int64_t)m1 * N;
  return gemm<true, BKROW, EPI, SEG>(a2, B, e2, M - m1, N, K, st);
}


constexpr float kLnEps = 1e-5f;

hipError_t launch_attn_fwd(const Geo& g, int dt, bool nhwc, const void* q, const void* k, const void* v,
                           const float* table, void* o, void* olo, float* lse, hipStream_t st);
hipError_t launch_attn_bwd(const Geo& g, int dt, bool nhwc, const void* q, const void* k, const void* v,
                           const void* o, const void* olo, const void* dout, const float* lse,
                           const float* table, void* dq, void* dk, void* dv, float* dtab, void* ws,
                           hipStream_t st);
size_t bwd_workspace(const Geo& g, int dt);

static hipError_t ln_stats(const void* x, float* mu, float* rs, int T, int C, hipStream_t st) {
  const int per = kRowThreads / 64;
  hipLaunchKernelGGL(ln_stats_kernel, dim3((T + per - 1) / per), dim3(kRowThreads), 0, st, (const bf16*)x, mu, rs,
                     T, C, kLnEps);
  return hipGetLastError();
}

static size_t al(size_t x) { return (x + 255) / 256 * 256; }

// Forward workspace: the folded QKV and fc1 weights and their per-output
// sums and constants.
struct FwdWs {
  size_t wq, wf, sq, cq, sf, cf, part, total;
};
static FwdWs fwd_ws(const Geo& g) {
  const size_t C = g.C;
  FwdWs w;
  size_t off = 0;
  w.wq = off; off += al(3 * C * C * 2);
  w.wf = off; off += al(4 * C * C * 2);
  w.sq = off; off += al(3 * C * 4);
  w.cq = off; off += al(3 * C * 4);
  w.sf = off; off += al(4 * C * 4);
  w.cf = off; off += al(4 * C * 4);
  w.part = off; off += al(split_floats(g.B * g.H * g.W, g.C, 4 * g.C) * 4);
  w.total = off;
  return w;
}
size_t block_fwd_workspace(const Geo& g) { return fwd_ws(g).total; }

hipError_t launch_block_fwd(const Geo& g, const void* x, const BlockParams& p, const float* table, void* x2,
                            const BlockSaved& s, void* wsv, hipStream_t st) {
  const int T = g.B * g.H * g.W, C = g.C;
  const FwdWs w = fwd_ws(g);
  char* ws = reinterpret_cast<char*>(wsv);
  bf16* wq = reinterpret_cast<bf16*>(ws + w.wq);
  bf16* wf = reinterpret_cast<bf16*>(ws + w.wf);
  float *sq = reinterpret_cast<float*>(ws + w.sq), *cq = reinterpret_cast<float*>(ws + w.cq);
  float *sf = reinterpret_cast<float*>(ws + w.sf), *cf = reinterpret_cast<float*>(ws + w.cf);
  hipError_t e;
  EpiArgs ep = {};
#define TERRA_TRY(x)                    \
  do {                                  \
    if ((e = (x)) != hipSuccess) return e; \
  } while (0)
  // LN1 statistics and both folded weights; qkv = LN1(x) W_qkv^T + b_qkv with
  // LN1 folded into the weights and the epilogue, written as Q, K, V (NHWC)
  {
    const int per = kRowThreads / 64;
    const int b0 = (T + per - 1) / per, b1 = b0 + (3 * C + 3) / 4;
    const FoldArgs f0 = {(const bf16*)p.w_qkv, p.ln1_g, p.ln1_b, p.b_qkv, wq, sq, cq, 3 * C};
    const FoldArgs f1 = {(const bf16*)p.w_fc1, p.ln2_g, p.ln2_b, p.b_fc1, wf, sf, cf, 4 * C};
    hipLaunchKernelGGL(block_prep_kernel, dim3(b1 + C), dim3(kRowThreads), 0, st, (const bf16*)x, s.mu1, s.rstd1, T,
                       C, kLnEps, f0, f1, b0, b1);
    TERRA_TRY(hipGetLastError());
  }
  ep.out[0] = (bf16*)s.q; ep.out[1] = (bf16*)s.k; ep.out[2] = (bf16*)s.v; ep.split = C;
  ep.mean = s.mu1; ep.rstd = s.rstd1; ep.lns = sq; ep.lnc = cq;
  TERRA_TRY((gemm<true, true, EPI_LN_QKV>(mat(x, C, T), mat(wq, C, 3 * C), ep, T, 3 * C, C, st)));
  // windowed attention with the route fused in
  TERRA_TRY(launch_attn_fwd(g, 1, true, s.q, s.k, s.v, table, s.o, nullptr, s.lse, st));
  // x1 = x + o W_p^T + b_p
  ep = EpiArgs{};
  ep.out[0] = (bf16*)s.x1; ep.split = C; ep.aux = (const bf16*)x; ep.bias = p.b_proj;
  TERRA_TRY((gemm<true, true, EPI_BIAS_RES>(mat(s.o, C, T), mat(p.w_proj, C, C), ep, T, C, C, st)));
  // h = LN2(x1) W_1^T + b_1 (LN2 folded), a = GELU(h)
  TERRA_TRY(ln_stats(s.x1, s.mu2, s.rstd2, T, C, st));
  ep = EpiArgs{};
  ep.out[0] = (bf16*)s.h; ep.split = 4 * C; ep.out2 = (bf16*)s.a;
  ep.mean = s.mu2; ep.rstd = s.rstd2; ep.lns = sf; ep.lnc = cf;
  TERRA_TRY((gemm<true, true, EPI_LN_GELU>(mat(s.x1, C, T), mat(wf, C, 4 * C), ep, T, 4 * C, C, st)));
  // x2 = x1 + a W_2^T + b_2
  ep = EpiArgs{};
  ep.out[0] = (bf16*)x2; ep.split = C; ep.aux = (const bf16*)s.x1; ep.bias = p.b_fc2;
  TERRA_TRY((gemm_rounds<true, EPI_BIAS_RES>(mat(s.a, 4 * C, T), mat(p.w_fc2, 4 * C, C), ep, T, C, 4 * C,
                                              reinterpret_cast<float*>(ws + w.part), st)));
#undef TERRA_TRY
  return hipSuccess;
}

// Form and token slices of a weight gradient dW[Nl][Kl] over T tokens.  The
// eight-wave form takes as many slices as fill two whole rounds of one
// workgroup per CU (a third, nearly empty round would leave most CUs idle
// for a whole slice), each of at least four stages.
static Plan wgrad_plan(int T, int Nl, int Kl) {
  const int tiles = ((Nl + kBM - 1) / kBM) * ((Kl + kBM - 1) / kBM);
  int n = (2 * kMaxCusBlock) / tiles;
  if ((T + n - 1) / n < 4 * kBK) n = (T + 4 * kBK - 1) / (4 * kBK);
  n = std::max(1, std::min(n, kMaxWgradSlices));
  Plan best = {8, n};
  double c = plan_cost(Nl, Kl, T, best);
  for (int ns = 1; ns <= kMaxSplit && (ns == 1 || T >= 4 * kBK * ns); ++ns) {
    const double d = plan_cost(Nl, Kl, T, {4, ns});
    if (d < c) { c = d; best = {4, ns}; }
  }
  return without_empty(best, T);
}

// For tests: waves and slices, 100 nw + ns, of a product and of a weight
// gradient.
int block_product_plan(int M, int N, int K, int max_split) {
  const Plan p = plan_product(M, N, K, max_split);
  return 100 * p.nw + p.ns;
}
int block_wgrad_plan(int T, int Nl, int Kl) {
  const Plan p = wgrad_plan(T, Nl, Kl);
  return 100 * p.nw + p.ns;
}

// Backward workspace layout (bytes, 256-aligned pieces).
struct BwdWs {
  size_t dh, dln, dx1, dO, dq, dk, dv, ln, wt, attn, wpart, cpart, lpart, total;
  int cslices, lnwaves, rows_per_wave, cpart_rows, lgroups;
};

// A pure function of the geometry: the attention part is sized for kMaxCus
// whatever device the call runs on.
static BwdWs block_ws(const Geo& geo) {
  Geo g = geo;
  g.cus = kMaxCus;
  BwdWs w;
  const size_t T = (size_t)g.B * g.H * g.W, C = g.C;
  w.cslices = 512;                       // row slices of the bias-gradient column sums
  w.cpart_rows = (int)((T + w.cslices - 1) / w.cslices);
  // waves of the LayerNorm backward: 4096, on small grids one per four rows
  // (with 4096 on 960 tokens the partials, 25 MB of zeros, were most of its
  // 19 us); above 256 of them, first-level groups of 32 for their sums
  w.lnwaves = T >= 16384 ? 4096 : (int)std::max<size_t>(64, (T / 4 + 31) / 32 * 32);
  w.rows_per_wave = (int)((T + w.lnwaves - 1) / w.lnwaves);
  w.lgroups = w.lnwaves > 256 ? w.lnwaves / 32 : 0;
  size_t off = 0;
  w.dh = off; off += al(T * 4 * C * 2);
  w.dln = off; off += al(T * C * 4);
  w.dx1 = off; off += al(T * C * 2);
  w.dO = off; off += al(T * C * 2);
  w.dq = off; off += al(T * C * 2);
  w.dk = off; off += al(T * C * 2);
  w.dv = off; off += al(T * C * 2);
  w.ln = off; off += al(T * C * 2);
  w.wt = off; off += al(12 * C * C * 2);  // transposed W_fc2, W_fc1, W_proj, W_qkv
  w.attn = off; off += al(bwd_workspace(g, 1));
  size_t wmax = 0;                       // largest slices x output of the block's weight gradients
  for (int i = 0; i < 4; ++i) {
    const int nl = i == 0 ? (int)C : (i == 1 ? 4 * (int)C : (i == 2 ? 3 * (int)C : (int)C));
    const int kl = i == 0 ? 4 * (int)C : (int)C;
    wmax = std::max(wmax, (size_t)wgrad_plan((int)T, nl, kl).ns * nl * kl);
  }
  wmax = std::max({wmax, split_floats((int)T, (int)C, 4 * (int)C), split_floats((int)T, (int)C, 3 * (int)C)});
  w.wpart = off; off += al(wmax * 4);
  // column-sum partials: the colsum slices, or the dh product's 2 rows a row tile
  w.cpart = off; off += al((size_t)std::max((size_t)w.cslices, 2 * ((T + kBS - 1) / kBS)) * 4 * C * 4);
  w.lpart = off; off += al((size_t)(w.lnwaves + w.lgroups) * 2 * C * 4);
  w.total = off;
  return w;
}

size_t block_bwd_workspace(const Geo& g) { return block_ws(g).total; }

static hipError_t slice_sum(const float* part, float* out, int64_t n, int nslice, hipStream_t st) {
  if (nslice >= 64) {
    hipLaunchKernelGGL(slice_sum4_kernel, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, st, part, out, out, n, n, n,
                       nslice);
  } else {
    hipLaunchKernelGGL(slice_sum_kernel, dim3((unsigned)((n + kRowThreads - 1) / kRowThreads)), dim3(kRowThreads), 0,
                       st, part, out, n, n, nslice);
  }
  return hipGetLastError();
}

// LayerNorm parameter gradients from the per-wave partials
// [wave][dgamma C | dbeta C]: with many waves first sums over groups of 32
// consecutive ones, then one sum over the groups (or the waves), in order.
static hipError_t ln_param_grads(const float* lpart, float* dgamma, float* dbeta, int C, const BwdWs& w,
                                 hipStream_t st) {
  const float* src = lpart;
  int n = w.lnwaves;
  if (w.lgroups > 0) {
    float* grp = const_cast<float*>(lpart) + (size_t)w.lnwaves * 2 * C;
    hipLaunchKernelGGL(group_sum_kernel, dim3((2 * C + kRowThreads - 1) / kRowThreads, w.lgroups), dim3(kRowThreads),
                       0, st, lpart, grp, 2 * C, w.lnwaves / w.lgroups);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    src = grp;
    n = w.lgroups;
  }
  hipLaunchKernelGGL(slice_sum4_kernel, dim3((2 * C + 63) / 64), dim3(256), 0, st, src, dgamma, dbeta, (int64_t)C,
                     (int64_t)2 * C, (int64_t)2 * C, n);
  return hipGetLastError();
}

static hipError_t colsum(const Mat& X, int ncols, float* part, float* out, const BwdWs& w, hipStream_t st) {
  if (X.rows <= kColDirect) {
    hipLaunchKernelGGL(colsum_direct_kernel, dim3(ncols / 64), dim3(256), 0, st, X, out);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(colsum_kernel, dim3((ncols / 8 + kRowThreads - 1) / kRowThreads, w.cslices), dim3(kRowThreads),
                     0, st, X, ncols, part, w.cpart_rows);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return slice_sum(part, out, ncols, w.cslices, st);
}

// Weight gradient dW[Nl][Kl] = dY^T Z over all tokens (dY: T x Nl, Z: T x Kl),
// in token slices, reduced in slice order.  LNB: Z = LN(z) applied while
// staging.

template <bool SEG>
static hipError_t wgrad(const Mat& dY, const Mat& Z, int T, int Nl, int Kl, float* dW, char* ws, const BwdWs& w,
                        hipStream_t st) {
  EpiArgs ep = {};
  float* part = reinterpret_cast<float*>(ws + w.wpart);
  const Plan p = wgrad_plan(T, Nl, Kl);
  ep.outf = p.ns > 1 ? part : dW;
  const hipError_t e = p.nw == 8 ? gemm_form<false, false, EPI_F32, SEG, 8>(dY, Z, ep, Nl, Kl, T, p.ns, st)
                                 : gemm_form<false, false, EPI_F32, SEG, 4>(dY, Z, ep, Nl, Kl, T, p.ns, st);
  if (e != hipSuccess || p.ns == 1) return e;
  return slice_sum(part, dW, (int64_t)Nl * Kl, p.ns, st);
}

// The three-part operand's buffer resource covers 2 segstride + T C
// elements; its byte offsets must stay below 2^31.
static bool seg_fits(int T, int C, int64_t segstride) {
  return (2 * segstride + (int64_t)T * C) * 2 < ((int64_t)1 << 31);
}

// dz = LayerNorm backward of dy (float32 or bf16) + dres, and the per-wave
// gain/shift partials, with the chunk count C needs.
template <typename DY>
static hipError_t ln_bwd(const DY* dy, const void* z, const float* mean, const float* rstd, const float* gamma,
                         const void* dres, void* dz, float* part, int T, int C, const BwdWs& w, hipStream_t st) {
  const dim3 grid(w.lnwaves / 4), block(kRowThreads);
  const bf16* zb = (const bf16*)z;
  const bf16* rb = (const bf16*)dres;
  bf16* ob = (bf16*)dz;
  switch ((C + 511) / 512) {
    case 1: hipLaunchKernelGGL((ln_bwd_kernel<DY, 1>), grid, block, 0, st, dy, zb, mean, rstd, gamma, rb, ob, part, T,
                               C, w.rows_per_wave); break;
    case 2: hipLaunchKernelGGL((ln_bwd_kernel<DY, 2>), grid, block, 0, st, dy, zb, mean, rstd, gamma, rb, ob, part, T,
                               C, w.rows_per_wave); break;
    case 3: hipLaunchKernelGGL((ln_bwd_kernel<DY, 3>), grid, block, 0, st, dy, zb, mean, rstd, gamma, rb, ob, part, T,
                               C, w.rows_per_wave); break;
    default: hipLaunchKernelGGL((ln_bwd_kernel<DY, 4>), grid, block, 0, st, dy, zb, mean, rstd, gamma, rb, ob, part,
                                T, C, w.rows_per_wave); break;
  }
  return hipGetLastError();
}

static hipError_t ln_apply(const void* z, const float* mu, const float* rs, const float* gamma, const float* beta,
                           bf16* out, int T, int C, hipStream_t st) {
  const int64_t n = (int64_t)T * (C / 8);
  hipLaunchKernelGGL(ln_apply_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const bf16*)z, mu, rs,
                     gamma, beta, out, T, C);
  return hipGetLastError();
}

hipError_t launch_block_bwd(const Geo& g, const void* dx2, const void* x, const BlockParams& p, const float* table,
                            const BlockSaved& s, void* dx, const BlockGrads& gr, float* dtable, void* wsv,
                            hipStream_t st) {
  const int T = g.B * g.H * g.W, C = g.C;
  const BwdWs w = block_ws(g);
  char* ws = reinterpret_cast<char*>(wsv);
  bf16* dh = reinterpret_cast<bf16*>(ws + w.dh);
  float* dln = reinterpret_cast<float*>(ws + w.dln);
  bf16* dlnb = reinterpret_cast<bf16*>(ws + w.dln);     // the same buffer holding bf16
  bf16* dx1 = reinterpret_cast<bf16*>(ws + w.dx1);
  bf16* dO = reinterpret_cast<bf16*>(ws + w.dO);
  bf16* dqkv[3] = {reinterpret_cast<bf16*>(ws + w.dq), reinterpret_cast<bf16*>(ws + w.dk),
                   reinterpret_cast<bf16*>(ws + w.dv)};
  float* cpart = reinterpret_cast<float*>(ws + w.cpart);
  float* lpart = reinterpret_cast<float*>(ws + w.lpart);
  bf16* lnb = reinterpret_cast<bf16*>(ws + w.ln);
  hipError_t e;
  EpiArgs ep = {};
#define TERRA_TRY(x)                    \
  do {                                  \
    if ((e = (x)) != hipSuccess) return e; \
  } while (0)
  // the weights in [N][K] order for the data-gradient products
  bf16* wt_fc2 = reinterpret_cast<bf16*>(ws + w.wt);        // [4C][C]
  bf16* wt_fc1 = wt_fc2 + (size_t)4 * C * C;                // [C][4C]
  bf16* wt_proj = wt_fc1 + (size_t)4 * C * C;               // [C][C]
  bf16* wt_qkv = wt_proj + (size_t)C * C;                   // [C][3C]
  {
    BwdPrep pr = {{(const bf16*)p.w_fc2, (const bf16*)p.w_fc1, (const bf16*)p.w_proj, (const bf16*)p.w_qkv},
                  {wt_fc2, wt_fc1, wt_proj, wt_qkv},
                  {C, 4 * C, C, 3 * C},
                  {4 * C, C, C, C},
                  {}};
    const int tl = C / 32;                                  // C is a multiple of 128
    pr.b[0] = 4 * tl * tl; pr.b[1] = 8 * tl * tl; pr.b[2] = 9 * tl * tl; pr.b[3] = 12 * tl * tl;
    const int64_t nln = ((int64_t)T * (C / 8) + 255) / 256;
    hipLaunchKernelGGL(block_bwd_prep_kernel, dim3((unsigned)(pr.b[3] + nln)), dim3(256), 0, st, pr,
                       (const bf16*)s.x1, s.mu2, s.rstd2, p.ln2_g, p.ln2_b, lnb, T, C);
    TERRA_TRY(hipGetLastError());
  }
  // x2 = x1 + a W2^T + b2:  dW2 = dx2^T a, db2 = colsum(dx2), dh = (dx2 W2) * GELU'(h)
  TERRA_TRY(wgrad<false>(mat(dx2, C, T), mat(s.a, 4 * C, T), T, C, 4 * C, gr.w_fc2, ws, w, st));
  TERRA_TRY(colsum(mat(dx2, C, T), C, cpart, gr.b_fc2, w, st));
  // db1 = colsum(dh) from the same epilogue: per-wave partial rows, then a
  // fixed-order sum of the two of each row tile
  ep.out[0] = dh; ep.split = 4 * C; ep.aux = (const bf16*)s.h; ep.colpart = cpart;
  TERRA_TRY((gemm<true, true, EPI_GELU_GRAD>(mat(dx2, C, T), mat(wt_fc2, C, 4 * C), ep, T, 4 * C, C, st)));
  {
    const int bm = plan_product(T, 4 * C, C, 1).nw == 8 ? kBM : kBS;      // the dh product's row tiles
    TERRA_TRY(slice_sum(cpart, gr.b_fc1, 4 * C, 2 * ((T + bm - 1) / bm), st));
  }
  // h = LN2(x1) W1^T + b1:  dW1 = dh^T LN2(x1), db1 = colsum(dh), dln2 = dh W1
  TERRA_TRY(wgrad<false>(mat(dh, 4 * C, T), mat(lnb, C, T), T, 4 * C, C, gr.w_fc1, ws, w, st));
  // dln2 in bf16, like the other gradients the products hand on
  ep = EpiArgs{};
  ep.out[0] = dlnb; ep.split = C;
  TERRA_TRY((gemm_rounds<true, EPI_BF16>(mat(dh, 4 * C, T), mat(wt_fc1, 4 * C, C), ep, T, C, 4 * C,
                                          reinterpret_cast<float*>(ws + w.wpart), st)));
  // dx1 = dx2 + LN2 backward
  TERRA_TRY(ln_bwd(dlnb, s.x1, s.mu2, s.rstd2, p.ln2_g, dx2, dx1, lpart, T, C, w, st));
  TERRA_TRY(ln_param_grads(lpart, gr.ln2_g, gr.ln2_b, C, w, st));
  // x1 = x + o Wp^T + bp:  dWp = dx1^T o, dbp = colsum(dx1), dO = dx1 Wp
  TERRA_TRY(wgrad<false>(mat(dx1, C, T), mat(s.o, C, T), T, C, C, gr.w_proj, ws, w, st));
  TERRA_TRY(colsum(mat(dx1, C, T), C, cpart, gr.b_proj, w, st));
  ep = EpiArgs{};
  ep.out[0] = dO; ep.split = C;
  TERRA_TRY((gemm<true, true, EPI_BF16>(mat(dx1, C, T), mat(wt_proj, C, C), ep, T, C, C, st)));
  // attention backward (route fused in)
  TERRA_TRY(launch_attn_bwd(g, 1, true, s.q, s.k, s.v, s.o, nullptr, dO, s.lse, table, dqkv[0], dqkv[1],
                            dqkv[2], dtable, ws + w.attn, st));
  // qkv = LN1(x) Wqkv^T + bqkv, one third (Q, K, V) at a time: rows
  // [iC, (i+1)C) of dWqkv = dY_i^T LN1(x), of dbqkv = colsum(dY_i), and
  // dln1 = sum_i dY_i Wqkv[iC:(i+1)C]
  TERRA_TRY(ln_apply(x, s.mu1, s.rstd1, p.ln1_g, p.ln1_b, lnb, T, C, st));
  // dQ, dK, dV sit at equal strides in the workspace: one T x 3C operand of
  // three parts, so that dWqkv is one product over all tokens and dln one
  // product over 3C (instead of three, two of them adding float32 results)
  Mat dy3 = mat(dqkv[0], C, T);
  dy3.segw = C;
  dy3.segstride = (int64_t)(w.dk - w.dq) / 2;
  const bool seg_w = (C % kBM == 0 || (wgrad_plan(T, 3 * C, C).nw == 4 && C % kBS == 0)) &&
                     seg_fits(T, C, dy3.segstride);
  const bool seg_d = C % kBK == 0 && seg_fits(T, C, dy3.segstride);
  if (seg_w) {
    TERRA_TRY(wgrad<true>(dy3, mat(lnb, C, T), T, 3 * C, C, gr.w_qkv, ws, w, st));
  }
  if (!seg_w) {
    for (int i = 0; i < 3; ++i)
      TERRA_TRY(wgrad<false>(mat(dqkv[i], C, T), mat(lnb, C, T), T, C, C, gr.w_qkv + (size_t)i * C * C, ws, w, st));
  }
  TERRA_TRY(colsum(dy3, 3 * C, cpart, gr.b_qkv, w, st));
  ep = EpiArgs{};
  if (seg_d) {
    ep.out[0] = dlnb; ep.split = C;
    TERRA_TRY((gemm_rounds<true, EPI_BF16, true>(dy3, mat(wt_qkv, 3 * C, C), ep, T, C, 3 * C,
                                                reinterpret_cast<float*>(ws + w.wpart), st)));
  } else {
    ep.outf = dln;
    for (int i = 0; i < 3; ++i) {
      const bf16* wi = reinterpret_cast<const bf16*>(p.w_qkv) + (size_t)i * C * C;
      if (i == 0) {
        TERRA_TRY((gemm<true, false, EPI_F32>(mat(dqkv[i], C, T), mat(wi, C, C), ep, T, C, C, st)));
      } else {
        TERRA_TRY((gemm<true, false, EPI_F32_ACC>(mat(dqkv[i], C, T), mat(wi, C, C), ep, T, C, C, st)));
      }
    }
  }
  // dx = dx1 + LN1 backward
  if (seg_d) {
    TERRA_TRY(ln_bwd(dlnb, x, s.mu1, s.rstd1, p.ln1_g, dx1, dx, lpart, T, C, w, st));
  } else {
    TERRA_TRY(ln_bwd(dln, x, s.mu1, s.rstd1, p.ln1_g, dx1, dx, lpart, T, C, w, st));
  }
  TERRA_TRY(ln_param_grads(lpart, gr.ln1_g, gr.ln1_b, C, w, st));
#undef TERRA_TRY
  return hipSuccess;
}

}  // namespace terra
