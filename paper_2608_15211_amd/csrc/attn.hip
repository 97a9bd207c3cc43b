// attn.hip - shifted-window multi-head self-attention for gfx950.
//
// The Swin blocks of the paper (Sec. IV-A, W-MSA / SW-MSA) attend inside
// each window of the window-major layout built by the token route
// (Sec. IV-D).  Per window and head:
//   S = Q K^T / sqrt(hd) + T[bin(q, k)],  masked pairs excluded,
//   P = softmax(S),  O = P V,  LSE = ln sum_k exp S
// and the backward
//   dV = P^T dO,  dP = dO V^T,  dS = P (dP - D),  D_q = sum_k P dP,
//   dQ = dS K / sqrt(hd),  dK = dS^T Q / sqrt(hd),  dT[bin] = sum dS.
//
// Kernel design (CDNA4, wave64):
// * QK^T, PV, dO V^T, dS K, dS^T Q and P^T dO run on the matrix cores
//   (32x32x16 bf16, or 32x32x2 fp32 for the fp32 path), fp32 accumulate.
// * A wave owns 32 queries (forward, dQ) or 32 keys (dK/dV).  The score
//   tile is produced TRANSPOSED where its rows must feed the next product
//   from registers: the result layout of one MFMA is then directly the
//   register operand of the next, with the contraction order permuted
//   consistently on the LDS side (no register shuffles).
// * K/V (forward, dQ) or Q/dO (dK/dV) tiles of 64 tokens are staged in LDS
//   by the whole workgroup, once row-major and once transposed where an
//   operand needs the token dimension as its contraction dimension.
// * Softmax runs in the log2 domain with an online max over key tiles; the
//   bias table of one head lives in LDS (pre-scaled by log2 e) and the mask
//   is a label compare per pair.
// * The bias-table gradient is summed per workgroup in LDS (one head per
//   workgroup, many windows per workgroup), written as per-workgroup
//   partials, and reduced in a fixed order by a second kernel.
#include <algorithm>
#include <type_traits>

#include "terra_common.h"
#include "terra_tile.h"

namespace terra {

// Window-resident path (attn_win.hip) for windows of at most 128 tokens.
bool win_fwd_ok(const Geo& g, bool bf16_);
bool win_bwd_ok(const Geo& g, bool bf16_);
int win_bwd_nslice(const Geo& g);
size_t win_fwd_lds(const Geo& g);
size_t win_bwd_lds(const Geo& g);
hipError_t launch_win_fwd(const Geo& g, bool nhwc, const void* q, const void* k, const void* v,
                          const float* table, void* o, float* lse, hipStream_t st);
hipError_t launch_win_bwd(const Geo& g, bool nhwc, const void* q, const void* k, const void* v,
                          const void* dout, const float* lse, const float* table, void* dq,
                          void* dk, void* dv, float* partial, int nslice, hipStream_t st);
// Fixed-order sum of the per-slice bias-gradient partials (dtab.hip).
hipError_t launch_dtab_reduce(const Geo& g, const float* partial, float* dtab, int nslice,
                              hipStream_t st);

constexpr int kThreads = 256;   // 4 waves
constexpr int kWaveQ = 32;      // queries (or keys) per wave
constexpr int kChunk = 128;     // queries (or keys) per workgroup
// Keys (or queries) per LDS tile: 64, or 32 for fp32 with head_dim 64 or 128
// (so that a staged tile set stays within 80 KB of LDS).
template <typename T, int HD> constexpr int tile_of() { return (sizeof(T) == 4 && HD >= 64) ? 32 : 64; }
constexpr int kPad = 8;         // LDS row padding, elements
constexpr int kLabBad = 0xFF;   // label of padding slots (never matches)

// Work item of a workgroup, one contiguous range of items per XCD: the hardware
// hands consecutive workgroups to the 8 XCDs in turn, and this puts the query
// chunks of one window and head, which stage the same K/V tiles, behind the
// same L2 (float32 forward -2 to -4 %; the eight-wave dQ kernel; measured no
// better or slower for the general dQ and the float32 dK/dV kernel, which keep
// the plain order).  The grid is rounded up to a multiple of 8 and the padding
// workgroups exit at once.
__device__ inline int xcd_item(int bid, int nblocks) { return (bid & 7) * (nblocks >> 3) + (bid >> 3); }
static inline int grid8(int n) { return (n + 7) & ~7; }
// The same for the 16-bit forward and dK/dV with one unit of `unit`
// consecutive items (the chunks of a window and head, and the heads that share
// a 128-byte line) per XCD in turn: contiguous ranges gave some XCDs the full
// windows and others the short ones of a ragged last row (25 rows of 24-row
// windows: dK/dV 233 -> 271 us).  TURN (dK/dV): each turn of eight units starts
// one XCD further, or a row of windows that is a whole number of turns puts
// its ragged last window on the same XCDs in every row (21 x 31 windows on 64 x
// 96 tokens, 12 heads of 32: 54 us, with it 42).  The forward measured 0.93 to
// 1.07 with it and keeps the plain turn.
template <bool TURN>
__device__ inline int xcd_unit_item(int bid, int unit) {
  const int idx = bid >> 3, u = idx / unit;
  return (u * 8 + ((TURN ? bid + u : bid) & 7)) * unit + (idx - u * unit);
}
static inline int unit_grid(int n, int unit) { return ((n + unit - 1) / unit + 7) / 8 * 8 * unit; }
// Up to two workgroups a CU, whole units would leave some XCDs short: single
// items then (240 workgroups of 768 tokens: forward 26 us in units of 12).
template <int HD>
static int xcd_unit(const Geo& g, int chunks) {
  return g.B * g.nwin * g.heads * chunks <= 2 * g.cus ? 1 : (HD == 32 ? 2 : 1) * chunks;
}

// Transposed tiles (head-dim rows e, token columns): row e starts at
// e * (kTile + kPad) plus 4 elements per group of 8 rows, so that the
// transposing staging stores of one instruction (8 rows of one chunk, the
// chunks 8 rows apart) fall in distinct LDS banks.
template <typename T, int HD>
__device__ __host__ constexpr int tr_row(int e) { return e * (tile_of<T, HD>() + kPad) + (e >> 3) * 4; }
template <typename T, int HD>
__device__ __host__ constexpr int tr_size() { return tr_row<T, HD>(HD); }

// Transposed copy of a tile: needed for fp32 only (16-bit tiles are read
// transposed straight from their row-major copy).
template <typename T, int HD>
__device__ __host__ constexpr int ttile_size() { return sizeof(T) == 2 ? 0 : tr_size<T, HD>(); }

template <typename T>
__device__ inline typename Operand<T>::type load_op_global(const T* p) {
  return *reinterpret_cast<const typename Operand<T>::type*>(p);
}
template <typename T>
__device__ inline typename Operand<T>::type zero_op() {
  typename Operand<T>::type z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = from_float<T>(0.0f);
  return z;
}
// Operand from an LDS row, 8 consecutive elements.
template <typename T>
__device__ inline typename Operand<T>::type load_op_lds(const T* p) {
  return *reinterpret_cast<const typename Operand<T>::type*>(p);
}
// Operand from an LDS row in the permuted slot order (two runs of 4).
template <typename T>
__device__ inline typename Operand<T>::type load_op_lds_perm(const T* row, int h) {
  typename Operand<T>::type o;
  const T* p0 = row + 4 * h;
  const T* p1 = row + 8 + 4 * h;
#pragma unroll
  for (int s = 0; s < 4; ++s) { o[s] = p0[s]; o[4 + s] = p1[s]; }
  return o;
}

// One staged tile of one tensor held in registers between its load from HBM
// and its store to LDS, so that the next tile's loads overlap the current
// tile's matrix work: thread t holds 16-byte chunks t, t+256, ... (row =
// chunk / chunks-per-row).
template <typename T, int HD>
struct TileRegs {
  static constexpr int kCpr = HD * (int)sizeof(T) / 16;
  static constexpr int kPer = tile_of<T, HD>() * kCpr / kThreads;
  uint4 r[kPer];
};

template <typename T, int HD, bool NHWC>
__device__ inline void tile_load(TileRegs<T, HD>& t, const T* __restrict__ src, const Geo& g,
                                 const WinTokens<NHWC>& wt, int r0, int n, int hoff) {
  constexpr int kCpr = TileRegs<T, HD>::kCpr;
#pragma unroll
  for (int u = 0; u < TileRegs<T, HD>::kPer; ++u) {
    const int idx = threadIdx.x + u * kThreads;
    const int rr = idx / kCpr, ch = idx % kCpr;
    const int row = r0 + rr;
    t.r[u] = make_uint4(0, 0, 0, 0);
    if (row < n)
      t.r[u] = *reinterpret_cast<const uint4*>(src + wt.tok(g, row) * g.C + hoff + ch * (16 / (int)sizeof(T)));
  }
}

// Element offsets (token index times C) of the window's n tokens, so that
// the staging of each later tile reads its row addresses from LDS instead of
// redoing the shifted-coordinate arithmetic per chunk (fused route only;
// window-major rows are consecutive).  The writes become visible to the
// other waves at the next barrier; the first tile is staged from its own
// arithmetic.
template <bool NHWC>
__device__ inline void tok_fill(uint32_t* tt, const Geo& g, const WinTokens<NHWC>& wt, int n) {
  if constexpr (NHWC)
    for (int t = threadIdx.x; t < n; t += kThreads) tt[t] = wt.tok(g, t) * (uint32_t)g.C;
}

// tile_load with the row offsets taken from the table.
template <typename T, int HD, bool NHWC>
__device__ inline void tile_load_tt(TileRegs<T, HD>& t, const T* __restrict__ src, const Geo& g,
                                    const WinTokens<NHWC>& wt, const uint32_t* tt, int r0, int n,
                                    int hoff) {
  if constexpr (!NHWC) {
    tile_load(t, src, g, wt, r0, n, hoff);
  } else {
    constexpr int kCpr = TileRegs<T, HD>::kCpr;
#pragma unroll
    for (int u = 0; u < TileRegs<T, HD>::kPer; ++u) {
      const int idx = threadIdx.x + u * kThreads;
      const int rr = idx / kCpr, ch = idx % kCpr;
      const int row = r0 + rr;
      t.r[u] = make_uint4(0, 0, 0, 0);
      if (row < n)
        t.r[u] = *reinterpret_cast<const uint4*>(src + tt[row] + hoff + ch * (16 / (int)sizeof(T)));
    }
  }
}

template <typename T, int HD, bool ROWMAJOR, bool TRANS>
__device__ inline void tile_store(const TileRegs<T, HD>& t, T* lds_rm, T* lds_tr) {
  constexpr int kCpr = TileRegs<T, HD>::kCpr;
  constexpr int kElemPerChunk = 16 / sizeof(T);
#pragma unroll
  for (int u = 0; u < TileRegs<T, HD>::kPer; ++u) {
    const int idx = threadIdx.x + u * kThreads;
    const int rr = idx / kCpr, ch = idx % kCpr;
    if (ROWMAJOR) *reinterpret_cast<uint4*>(lds_rm + rr * (HD + kPad) + ch * kElemPerChunk) = t.r[u];
    if (TRANS) {
      const T* e = reinterpret_cast<const T*>(&t.r[u]);
#pragma unroll
      for (int x = 0; x < kElemPerChunk; ++x) lds_tr[tr_row<T, HD>(ch * kElemPerChunk + x) + rr] = e[x];
    }
  }
}

// Label/bias-offset word of in-window token t (t < n), or of a pad slot.
__device__ inline int token_info(const Geo& g, int i, int j, int cols, int t, int n) {
  if (t >= n) return kLabBad << 24;
  const int a = fast_div(t, cols, win_rcols(g, j));
  const int c = t - a * cols;
  const int lab = row_label(g, i * g.wh + a) | col_label(g, j * g.ww + c);
  return (a * g.bstride + c) | (lab << 24);
}

// bias_init with each key's bias offset also held as a byte offset, knb[k]
// = 4 x (offset of key k): one group of four keys then costs one address add
// from tabq, the lane's row of the reversed table in bytes.  Labels still
// come from kinfo, and an excluded pair reads its bin (always inside the
// table) and is replaced by -inf.
template <bool QUAD, bool MASK>
__device__ inline f32x16 bias_init_nb(const int* kinfo, const int* knb, const char* tabq, int kb,
                                      int half, int qlab) {
  f32x16 c;
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4) {
    const int kk = 32 * kb + 8 * g4 + 4 * half;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int kx = QUAD ? kk : kk + x;
      c[4 * g4 + x] = reinterpret_cast<const float*>(tabq + knb[kx])[QUAD ? x : 0];
      if (MASK && (kinfo[kx] >> 24) != qlab) c[4 * g4 + x] = -INFINITY;
    }
  }
  return c;
}

// The same with the labels in an array of their own.
template <bool QUAD, bool MASK>
__device__ inline f32x16 bias_init_lab(const int* klabs, const int* knb, const char* tabq, int kb,
                                       int half, int qlab) {
  f32x16 c;
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4) {
    const int kk = 32 * kb + 8 * g4 + 4 * half;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int kx = QUAD ? kk : kk + x;
      c[4 * g4 + x] = reinterpret_cast<const float*>(tabq + knb[kx])[QUAD ? x : 0];
      if (MASK && klabs[kx] != qlab) c[4 * g4 + x] = -INFINITY;
    }
  }
  return c;
}

// The key-major form (lane = key, registers = queries of query block QB):
// qnb[t] = 4 x (offset of query t), tabk the lane's row of the forward-order
// table in bytes.
template <bool QUAD, bool MASK>
__device__ inline f32x16 bias_init_t_nb(const int* qinfo, const int* qnb, const char* tabk, int qb,
                                        int half, int klab) {
  f32x16 c;
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4) {
    const int qq = 32 * qb + 8 * g4 + 4 * half;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int qx = QUAD ? qq : qq + x;
      c[4 * g4 + x] = reinterpret_cast<const float*>(tabk + qnb[qx])[QUAD ? x : 0];
      if (MASK && (qinfo[qx] >> 24) != klab) c[4 * g4 + x] = -INFINITY;
    }
  }
  return c;
}

// ---------------------------------------------------------------------------
// Forward.  Grid: B * nwin * heads * nqc workgroups (nqc query chunks of 128
// per window, empty chunks of small windows exit at once).  The bias enters
// the score accumulator before the QK^T product (table times sqrt(hd) in
// reversed bin order, -inf entries for excluded pairs), so each score costs
// one multiply-add and one exp2 outside the matrix cores.  float32 only: the
// 16-bit types have fwd16_kernel.
// ---------------------------------------------------------------------------
template <typename T, int HD, bool NHWC, bool QUAD>
__global__ __launch_bounds__(kThreads) void fwd_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const float* __restrict__ table, T* __restrict__ o,
    float* __restrict__ lse, Geo g, int nqc, float scale_log2) {
  constexpr int kTile = tile_of<T, HD>();
  extern __shared__ __align__(16) char smem[];
  T* kt = reinterpret_cast<T*>(smem);                          // [kTile][HD+kPad]
  T* vt = kt + kTile * (HD + kPad);                            // V^T
  int* kinfo = reinterpret_cast<int*>(vt + tr_size<T, HD>());
  float* tab = reinterpret_cast<float*>(kinfo + kTile);        // [nbins+4], reversed
  uint32_t* tt = reinterpret_cast<uint32_t*>(tab + g.nbins + 4);   // [wh*ww] token offsets

  int bid = xcd_item(blockIdx.x, gridDim.x);
  if (bid >= g.B * g.nwin * g.heads * nqc) return;
  const int qc = bid % nqc; bid /= nqc;
  const int h = bid % g.heads; bid /= g.heads;
  const int w = bid % g.nwin;
  const int b = bid / g.nwin;
  const int i = w / g.Mw, j = w - (w / g.Mw) * g.Mw;
  const int cols = win_cols(g, j);
  const int n = win_rows(g, i) * cols;
  const int q0 = qc * kChunk;
  if (q0 >= n) return;
  const WinTokens<NHWC> wt(g, b, i, j);
  const int hoff = h * HD;

  const float bscale = sqrtf((float)HD);
  for (int x = threadIdx.x; x < g.nbins + 4; x += kThreads)
    tab[x] = x < g.nbins ? table[(g.nbins - 1 - x) * g.heads + h] * bscale : -INFINITY;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int qi = q0 + wave * kWaveQ + col;
  const bool qvalid = qi < n;
  // waves whose 32 queries all lie past the window's end (last chunk of a
  // window that is not a multiple of 128 tokens) skip the matrix work
  const bool wactive = q0 + wave * kWaveQ < n;
  const int qinf = token_info(g, i, j, cols, qvalid ? qi : 0, n);
  const int qlab = qinf >> 24;
  const int qrev = g.nbins - 1 - ((qinf & 0xFFFFFF) + (g.wh - 1) * g.bstride + (g.ww - 1));
  const bool mask = window_has_labels(g, i, j) || (n % kTile) != 0;

  typename Operand<T>::type qop[HD / 16];
#pragma unroll
  for (int c = 0; c < HD / 16; ++c)
    qop[c] = qvalid ? load_op_global<T>(q + wt.tok(g, qi) * g.C + hoff + 16 * c + 8 * half)
                    : zero_op<T>();

  f32x16 oacc[HD / 32];
#pragma unroll
  for (int eb = 0; eb < HD / 32; ++eb) oacc[eb] = f32x16{};
  float m_run = -1e30f, l_run = 0.0f;     // running max (log2 units) and sum

  // K, V tiles go HBM -> registers -> LDS, one tile ahead up to head dim 64
  constexpr bool kPrefetch = HD <= 64;
  TileRegs<T, HD> rk, rv;
  if (kPrefetch) {
    tile_load(rk, k, g, wt, 0, n, hoff);
    tile_load(rv, v, g, wt, 0, n, hoff);
  }
  tok_fill(tt, g, wt, n);
  if (!kPrefetch && NHWC) lds_barrier();   // the first tile comes from the table too
  for (int k0 = 0; k0 < n; k0 += kTile) {
    if (!kPrefetch) {
      tile_load_tt(rk, k, g, wt, tt, k0, n, hoff);
      tile_load_tt(rv, v, g, wt, tt, k0, n, hoff);
    }
    lds_barrier();
    tile_store<T, HD, true, false>(rk, kt, nullptr);
    tile_store<T, HD, false, true>(rv, nullptr, vt);
    if (threadIdx.x < kTile) kinfo[threadIdx.x] = token_info(g, i, j, cols, k0 + threadIdx.x, n);
    lds_barrier();
    if (kPrefetch && k0 + kTile < n) {
      tile_load_tt(rk, k, g, wt, tt, k0 + kTile, n, hoff);
      tile_load_tt(rv, v, g, wt, tt, k0 + kTile, n, hoff);
    }
    if (!wactive) continue;     // staging and barriers only

    f32x16 s[kTile / 32];
    float mloc = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < kTile / 32; ++kb) {
      s[kb] = mask ? bias_init<QUAD, true>(kinfo, tab, kb, half, qrev, qlab, g.nbins)
                   : bias_init<QUAD, false>(kinfo, tab, kb, half, qrev, qlab, g.nbins);
#pragma unroll
      for (int c = 0; c < HD / 16; ++c)
        mma16(s[kb], load_op_lds<T>(kt + (kb * 32 + col) * (HD + kPad) + 16 * c + 8 * half), qop[c]);
#pragma unroll
      for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, s[kb][r]);
    }
    mloc = halves_max(mloc);
    // The running maximum moves (and O and the sum are rescaled) only when
    // some query of the wave sees a score more than 2^8 above it: between
    // moves the weights stay below 256, which the fp32 sums carry as exactly
    // as weights below 1.
    const float mt = mloc * scale_log2;
    if (__builtin_amdgcn_ballot_w64(mt > m_run + 8.0f) != 0) {
      const float mnew = fmaxf(m_run, mt);
      const float alpha = exp2f(m_run - mnew);
      m_run = mnew;
      l_run *= alpha;
#pragma unroll
      for (int eb = 0; eb < HD / 32; ++eb) oacc[eb] *= alpha;
    }
#pragma unroll
    for (int kb = 0; kb < kTile / 32; ++kb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(s[kb][r] * scale_log2 - m_run);
        s[kb][r] = p;
        l_run += p;
      }
    }
#pragma unroll
    for (int eb = 0; eb < HD / 32; ++eb) {
#pragma unroll
      for (int kb = 0; kb < kTile / 32; ++kb) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const T* row = vt + tr_row<T, HD>(eb * 32 + col) + kb * 32 + 16 * c;
          mma16(oacc[eb], load_op_lds_perm<T>(row, half), pack8<T>(s[kb], 8 * c));
        }
      }
    }
  }
  l_run = halves_sum(l_run);
  if (!qvalid) return;
  const float inv = 1.0f / l_run;
  T* orow = o + wt.tok(g, qi) * g.C + hoff;
#pragma unroll
  for (int eb = 0; eb < HD / 32; ++eb) {
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
      const int e = eb * 32 + 8 * grp + 4 * half;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        orow[e + x] = from_float<T>(oacc[eb][4 * grp + x] * inv);
      }
    }
  }
  if (half == 0) lse[wt.lse_at(g, h, qi)] = (m_run + __log2f(l_run)) * kLn2;
}

// What the bias bins' fold (add_bins) needs to know of a lane: runs are lanes
// of one 32-lane half holding consecutive queries of one window row.
struct BinFold {
  bool on;               // every window width is a multiple of 4 (uniform)
  int run, rest;         // lanes before and after this one in its run
  float fnext;           // 1: lane l+1 is in the run, and this lane may pass to it
  float fkeep;           // 1: one of the run's first three
  __device__ BinFold(const Geo& g, int j, int cols, int qi, int col)
      : on((g.ww % 4 == 0) && (g.W % g.ww) % 4 == 0) {
    const int cq = qi - fast_div(qi, cols, win_rcols(g, j)) * cols;
    run = cq < col ? cq : col;
    rest = (cols - 1 - cq) < (31 - col) ? (cols - 1 - cq) : (31 - col);
    fnext = rest > 0 ? 1.0f : 0.0f;
    fkeep = run < 3 ? 1.0f : 0.0f;
  }
};

// Bias bins of one key tile: a wave adds dsb into the copy behind qbins (bin
// of (this lane's query, key kk): qbins - knb[kk] in bytes), and the two lane
// halves add with separate instructions.  Within one half, lanes hold distinct
// queries of the same key, hence distinct bins, so the additions are plain
// read-modify-writes (an LDS float atomic costs about three clocks per lane,
// some 170 times a store) and every bin receives them in program order; lanes
// with nothing to add (padding queries, excluded pairs) stay out.  When every
// window width is a multiple of 4, registers 4g..4g+3 hold four consecutive
// keys k..k+3 of one window row and (q, k+x), (q+1, k+x+1) share a bin.
// Within a run of consecutive lanes holding consecutive queries of one window
// row, a DPP chain towards lower lanes folds each group into one value (bin of
// (q, k)); the pairs it cannot reach (fewer than x lanes before q in the run)
// move towards higher lanes into the run's first three lanes (bin of
// (q', k+3)), and the few that would leave a run shorter than three lanes are
// added on their own.
// full: every query of the wave and every key of the tile is a window token.
template <int KB, typename NB>
__device__ __forceinline__ void add_bins(const f32x16 (&dsb)[KB], char* qbins, const NB* knb, const BinFold& bf,
                                         bool full, int half) {
  auto bin = [&](int kk) -> float& { return *reinterpret_cast<float*>(qbins - knb[kk]); };
  if (bf.on) {
    float fa[KB][4], fb[KB][4];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const float d0 = dsb[kb][4 * g4], d1 = dsb[kb][4 * g4 + 1];
        const float d2 = dsb[kb][4 * g4 + 2], d3 = dsb[kb][4 * g4 + 3];
        float f = d3;
        f = d2 + bf.fnext * dpp_lane<kDppNext>(f);
        f = d1 + bf.fnext * dpp_lane<kDppNext>(f);
        fa[kb][g4] = d0 + bf.fnext * dpp_lane<kDppNext>(f);
        const float p1 = dpp_lane<kDppWavePrev>(d2 * bf.fnext);
        const float p2 = dpp_lane<kDppWavePrev>(dpp_lane<kDppWavePrev>(d1 * bf.fnext) * bf.fnext);
        fb[kb][g4] = bf.fkeep * (d3 + p1 + p2);
      }
    // One update of this lane: the folded pair sums of key block kb,
    // group g4 (fa at (q, k), fb at (q, k+3)).
    auto upd = [&](int kb, int g4, float va, float vb) {
      const int kk = kb * 32 + 8 * g4 + 4 * half;
      if (va != 0.0f) bin(kk) += va;
      if (vb != 0.0f) bin(kk + 3) += vb;
    };
    if constexpr (KB == 2) {
      // Both halves update with one instruction when their keys are at
      // least 32 tokens apart: the 32 queries of a half are consecutive
      // tokens, so (q, k) and (q', k') share a bin only if |k - k'| =
      // |q - q'| < 32.  Half 0 takes block 0 group t while half 1 takes
      // block 1 group t (keys 32 + 4 or more apart), then half 0 takes
      // block 1 group t while half 1 takes block 0 group t - 1 (36 or
      // more), and the two updates left over go alone.
      if (full) {
        // Every query of the wave and every key of the tile is a window
        // token: the updates need no guard (adding 0 to a bin that no
        // other lane of the instruction touches changes nothing), and
        // the key words are read before the first update.  Word index of
        // this lane's group: 36 half + 8t in the first round, 32 - 36 half
        // + 8t in the second, 32 (half 0) or 28 (half 1) left over.
        float* w1[4][2];
        float* w2[3][2];
        float* wl[2];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int kk = 36 * half + 8 * t;
          w1[t][0] = &bin(kk);
          w1[t][1] = &bin(kk + 3);
        }
#pragma unroll
        for (int t = 1; t < 4; ++t) {
          const int kk = 32 - 36 * half + 8 * t;
          w2[t - 1][0] = &bin(kk);
          w2[t - 1][1] = &bin(kk + 3);
        }
        {
          const int kk = half ? 28 : 32;
          wl[0] = &bin(kk);
          wl[1] = &bin(kk + 3);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          *w1[t][0] += half ? fa[1][t] : fa[0][t];
          *w1[t][1] += half ? fb[1][t] : fb[0][t];
        }
#pragma unroll
        for (int t = 1; t < 4; ++t) {
          *w2[t - 1][0] += half ? fa[0][t - 1] : fa[1][t];
          *w2[t - 1][1] += half ? fb[0][t - 1] : fb[1][t];
        }
        if (half == 0) { *wl[0] += fa[1][0]; *wl[1] += fb[1][0]; }
        __builtin_amdgcn_wave_barrier();
        if (half == 1) { *wl[0] += fa[0][3]; *wl[1] += fb[0][3]; }
        __builtin_amdgcn_wave_barrier();
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int kb = half, gt = t;
          upd(kb, gt, half ? fa[1][t] : fa[0][t], half ? fb[1][t] : fb[0][t]);
        }
#pragma unroll
        for (int t = 1; t < 4; ++t) {
          const int kb = 1 - half, gt = t - half;
          upd(kb, gt, half ? fa[0][t - 1] : fa[1][t], half ? fb[0][t - 1] : fb[1][t]);
        }
        if (half == 0) upd(1, 0, fa[1][0], fb[1][0]);
        __builtin_amdgcn_wave_barrier();
        if (half == 1) upd(0, 3, fa[0][3], fb[0][3]);
        __builtin_amdgcn_wave_barrier();
      }
    } else {
#pragma unroll 1
      for (int hh = 0; hh < 2; ++hh) {
        if (half == hh) {
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) upd(0, g4, fa[0][g4], fb[0][g4]);
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
    // pairs of runs shorter than three lanes that the fold left out
    if (__builtin_amdgcn_ballot_w64((bf.run < 1 && bf.rest < 2) || (bf.run < 2 && bf.rest < 1)) != 0) {
#pragma unroll 1
      for (int hh = 0; hh < 2; ++hh) {
        if (half == hh) {
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
              const int kk = kb * 32 + 8 * g4 + 4 * half;
#pragma unroll
              for (int x = 1; x < 3; ++x)
                if (bf.run < x && bf.rest < 3 - x && dsb[kb][4 * g4 + x] != 0.0f)
                  bin(kk + x) += dsb[kb][4 * g4 + x];
            }
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
  } else {
#pragma unroll 1
    for (int hh = 0; hh < 2; ++hh) {
      if (half == hh) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            if (dsb[kb][r] != 0.0f) bin(kb * 32 + acc_row(r, half)) += dsb[kb][r];
          }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// ---------------------------------------------------------------------------
// Backward, step 1: D, dQ and the bias-table partials.  One head per
// workgroup; the workgroup walks items (image, window, query chunk)
// slice, slice + nslice, ... in a fixed order and accumulates dT in LDS.
// Per item, D_q = sum_k P dP = <dO_q, O_q> (O unrounded) is formed first
// and stored for the dK/dV kernel: from the forward's O and its rounding
// residual O_lo when the caller kept it (olo not null), else by a first
// sweep over the key tiles in fp32.  The stored 16-bit O alone is not
// enough: D's rounding error, alike for every key of a query, adds up over
// the windows in the bias-table gradient.  The (second) sweep forms dS, dQ
// and the bias bins.
// ---------------------------------------------------------------------------
template <typename T, int HD, bool NHWC, bool QUAD, bool RES>
__global__ __launch_bounds__(kThreads, 2) void bwd_dq_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const T* __restrict__ o, const T* __restrict__ olo,
    const T* __restrict__ dout, const float* __restrict__ lse, float* __restrict__ D,
    const float* __restrict__ table, T* __restrict__ dq, float* __restrict__ partial,
    Geo g, int nqc, int nslice, float scale_log2, float scale) {
  constexpr int kTile = tile_of<T, HD>();
  constexpr int kTE = kTile * (HD + kPad);            // elements of one staged tile
  // RES: every tile of the window stays in LDS for the whole item (nt tiles)
  const int nt = RES ? (g.wh * g.ww + kTile - 1) / kTile : 1;
  extern __shared__ __align__(16) char smem[];
  T* kt0 = reinterpret_cast<T*>(smem);                // K  nt x [kTile][HD+kPad]
  T* vr0 = kt0 + nt * kTE;                            // V  nt x [kTile][HD+kPad]
  T* ktt = vr0 + nt * kTE;                            // K^T (transposed tile, fp32)
  // nt x {[kTile] label/offset words, [kTile] 4 x offset}
  int* kinfo0 = reinterpret_cast<int*>(ktt + ttile_size<T, HD>());
  float* tab = reinterpret_cast<float*>(kinfo0 + 2 * nt * kTile);   // [nbins+4], reversed
  float* dtab = tab + g.nbins + 4;                    // [4][nbins], one per wave
  // [wh*ww] token offsets of the current item.  One buffer serves: the last
  // read of an item (the prefetch of its last tile) comes before the
  // barriers of that tile, which every wave passes before the next fill.
  uint32_t* tt = reinterpret_cast<uint32_t*>(dtab + 4 * g.nbins);

  const int h = blockIdx.x / nslice;
  const int slice = blockIdx.x - h * nslice;
  const int hoff = h * HD;
  const float bscale = sqrtf((float)HD);
  for (int x = threadIdx.x; x < g.nbins + 4; x += kThreads)
    tab[x] = x < g.nbins ? table[(g.nbins - 1 - x) * g.heads + h] * bscale : -INFINITY;
  for (int x = threadIdx.x; x < 4 * g.nbins; x += kThreads) dtab[x] = 0.0f;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int nitems = g.B * g.nwin * nqc;

  for (int it = slice; it < nitems; it += nslice) {
    const int qc = it % nqc;
    const int w = (it / nqc) % g.nwin;
    const int b = it / (nqc * g.nwin);
    const int i = w / g.Mw, j = w - (w / g.Mw) * g.Mw;
    const int cols = win_cols(g, j);
    const int n = win_rows(g, i) * cols;
    const int q0 = qc * kChunk;
    if (q0 >= n) continue;
    const WinTokens<NHWC> wt(g, b, i, j);
    const int qi = q0 + wave * kWaveQ + col;
    const bool qvalid = qi < n;
    const bool wactive = q0 + wave * kWaveQ < n;   // else staging and barriers only
    const int qinf = token_info(g, i, j, cols, qvalid ? qi : 0, n);
    const int qlab = qinf >> 24;
    const int qoff = (qinf & 0xFFFFFF) + (g.wh - 1) * g.bstride + (g.ww - 1);
    const int qrev = g.nbins - 1 - qoff;
    const char* tabq = reinterpret_cast<const char*>(tab + qrev);
    const int64_t lidx = wt.lse_at(g, h, qvalid ? qi : 0);
    // +inf for padding queries: their P is exactly 0
    const float lse2 = qvalid ? lse[lidx] * kLog2e : INFINITY;
    const bool mask = window_has_labels(g, i, j) || (n % kTile) != 0;

    typename Operand<T>::type qop[HD / 16], dop[HD / 16];
#pragma unroll
    for (int c = 0; c < HD / 16; ++c) {
      qop[c] = qvalid ? load_op_global<T>(q + wt.tok(g, qi) * g.C + hoff + 16 * c + 8 * half)
                      : zero_op<T>();
      dop[c] = qvalid ? load_op_global<T>(dout + wt.tok(g, qi) * g.C + hoff + 16 * c + 8 * half)
                      : zero_op<T>();
    }
    // D_q, then the sweep.  The K, V tiles go HBM -> registers -> LDS; up to
    // head dim 64 each tile's loads are issued while the previous tile
    // computes (after the last tile of the D sweep, or straight after these
    // first loads when D comes from O, come the first tiles of the main
    // sweep); at head dim 128 the registers this holds would halve the
    // occupancy.
    constexpr bool kPrefetch = HD <= 64;
    TileRegs<T, HD> rk, rv;
    if constexpr (RES) {
      // all tiles of the window into LDS once per item (each tile's loads
      // issued before the previous tile is stored); both sweeps then read
      // them without staging or barriers
      tile_load(rk, k, g, wt, 0, n, hoff);
      tile_load(rv, v, g, wt, 0, n, hoff);
      lds_barrier();                  // the previous item is done with the tiles
      for (int t0 = 0; t0 < n; t0 += kTile) {
        TileRegs<T, HD> nk = rk, nv = rv;
        if (t0 + kTile < n) {
          tile_load(nk, k, g, wt, t0 + kTile, n, hoff);
          tile_load(nv, v, g, wt, t0 + kTile, n, hoff);
        }
        const int tix = t0 / kTile;
        tile_store<T, HD, true, false>(rk, kt0 + tix * kTE, nullptr);
        tile_store<T, HD, true, false>(rv, vr0 + tix * kTE, nullptr);
        if (threadIdx.x < kTile) {
          const int inf = token_info(g, i, j, cols, t0 + threadIdx.x, n);
          kinfo0[tix * 2 * kTile + threadIdx.x] = inf;
          kinfo0[tix * 2 * kTile + kTile + threadIdx.x] = 4 * (inf & 0xFFFFFF);
        }
        rk = nk;
        rv = nv;
      }
      lds_barrier();
    } else if (kPrefetch) {
      tile_load(rk, k, g, wt, 0, n, hoff);
      tile_load(rv, v, g, wt, 0, n, hoff);
    }
    if constexpr (!RES) {
      tok_fill(tt, g, wt, n);
      if (!kPrefetch && NHWC) lds_barrier();   // the first tile comes from the table too
    }
    float dsum = 0.0f;
    if (olo != nullptr) {
      // D from the forward's output: the two halves of a lane pair hold
      // alternate 8-element runs of the query's row, like dop
      if (qvalid) {
        const T* orow = o + wt.tok(g, qi) * g.C + hoff;
        const T* lrow = olo + wt.tok(g, qi) * g.C + hoff;
#pragma unroll
        for (int c = 0; c < HD / 16; ++c) {
          const auto ov = load_op_global<T>(orow + 16 * c + 8 * half);
          const auto lv = load_op_global<T>(lrow + 16 * c + 8 * half);
#pragma unroll
          for (int x = 0; x < 8; ++x)
            dsum += to_float<T>(dop[c][x]) * (to_float<T>(ov[x]) + to_float<T>(lv[x]));
        }
      }
    } else for (int k0 = 0; k0 < n; k0 += kTile) {
      const int tix = RES ? k0 / kTile : 0;
      T* kt = kt0 + tix * kTE;
      T* vr = vr0 + tix * kTE;
      int* kinfo = kinfo0 + tix * 2 * kTile;
      int* knb = kinfo + kTile;
      if constexpr (!RES) {
        if (!kPrefetch) {
          tile_load_tt(rk, k, g, wt, tt, k0, n, hoff);
          tile_load_tt(rv, v, g, wt, tt, k0, n, hoff);
        }
        lds_barrier();
        tile_store<T, HD, true, false>(rk, kt, nullptr);
        tile_store<T, HD, true, false>(rv, vr, nullptr);
        if (threadIdx.x < kTile) {
          const int inf = token_info(g, i, j, cols, k0 + threadIdx.x, n);
          kinfo[threadIdx.x] = inf;
          knb[threadIdx.x] = 4 * (inf & 0xFFFFFF);
        }
        lds_barrier();
        if (kPrefetch) {
          const int nk0 = k0 + kTile < n ? k0 + kTile : 0;
          tile_load_tt(rk, k, g, wt, tt, nk0, n, hoff);
          tile_load_tt(rv, v, g, wt, tt, nk0, n, hoff);
        }
      }
      if (!wactive) continue;
#pragma unroll
      for (int kb = 0; kb < kTile / 32; ++kb) {
        f32x16 s = mask ? bias_init_nb<QUAD, true>(kinfo, knb, tabq, kb, half, qlab)
                        : bias_init_nb<QUAD, false>(kinfo, knb, tabq, kb, half, qlab);
        f32x16 dp = f32x16{};
#pragma unroll
        for (int c = 0; c < HD / 16; ++c) {
          mma16(s, load_op_lds<T>(kt + (kb * 32 + col) * (HD + kPad) + 16 * c + 8 * half), qop[c]);
          mma16(dp, load_op_lds<T>(vr + (kb * 32 + col) * (HD + kPad) + 16 * c + 8 * half), dop[c]);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r)
          dsum += __builtin_amdgcn_exp2f(s[r] * scale_log2 - lse2) * dp[r];
      }
    }
    const float Dq = halves_sum(dsum);
    if (qvalid && half == 0) D[lidx] = Dq;

    // main sweep: dS, dQ, bias bins
    const BinFold bf(g, j, cols, qi, col);
    f32x16 dqacc[HD / 32];
#pragma unroll
    for (int eb = 0; eb < HD / 32; ++eb) dqacc[eb] = f32x16{};

    for (int k0 = 0; k0 < n; k0 += kTile) {
      const int tix = RES ? k0 / kTile : 0;
      T* kt = kt0 + tix * kTE;
      T* vr = vr0 + tix * kTE;
      int* kinfo = kinfo0 + tix * 2 * kTile;
      int* knb = kinfo + kTile;
      if constexpr (!RES) {
        if (!kPrefetch) {
          tile_load_tt(rk, k, g, wt, tt, k0, n, hoff);
          tile_load_tt(rv, v, g, wt, tt, k0, n, hoff);
        }
        lds_barrier();
        tile_store<T, HD, true, sizeof(T) == 4>(rk, kt, ktt);
        tile_store<T, HD, true, false>(rv, vr, nullptr);
        if (threadIdx.x < kTile) {
          const int inf = token_info(g, i, j, cols, k0 + threadIdx.x, n);
          kinfo[threadIdx.x] = inf;
          knb[threadIdx.x] = 4 * (inf & 0xFFFFFF);
        }
        lds_barrier();
        if (kPrefetch && k0 + kTile < n) {
          tile_load_tt(rk, k, g, wt, tt, k0 + kTile, n, hoff);
          tile_load_tt(rv, v, g, wt, tt, k0 + kTile, n, hoff);
        }
      }
      if (!wactive) continue;
      // Head dim 64: the S and dP products of every key block of the tile
      // first, then per block dS and dQ += dS K, so that one block's exp
      // runs while the next block's products are on the matrix cores; each
      // block's K and V operands are read from LDS before its bias (dQ
      // kernel -3 % at 576-token windows).  Otherwise one block at a time:
      // at head dim 128 the held operands and accumulators would spill, and
      // at head dim 32 they would cost the third resident wave per SIMD.
      constexpr bool kHold = HD == 64;
      f32x16 dsb[kTile / 32];
      if constexpr (kHold) {
        f32x16 sb[kTile / 32];
#pragma unroll
        for (int kb = 0; kb < kTile / 32; ++kb) {
          typename Operand<T>::type kop_[HD / 16], vop_[HD / 16];
#pragma unroll
          for (int c = 0; c < HD / 16; ++c) {
            kop_[c] = load_op_lds<T>(kt + (kb * 32 + col) * (HD + kPad) + 16 * c + 8 * half);
            vop_[c] = load_op_lds<T>(vr + (kb * 32 + col) * (HD + kPad) + 16 * c + 8 * half);
          }
          __builtin_amdgcn_sched_barrier(0);
          sb[kb] = mask ? bias_init_nb<QUAD, true>(kinfo, knb, tabq, kb, half, qlab)
                        : bias_init_nb<QUAD, false>(kinfo, knb, tabq, kb, half, qlab);
#pragma unroll
          for (int r = 0; r < 16; ++r) dsb[kb][r] = -Dq;      // dP - D straight from the product
#pragma unroll
          for (int c = 0; c < HD / 16; ++c) {
            mma16(sb[kb], kop_[c], qop[c]);
            mma16(dsb[kb], vop_[c], dop[c]);
          }
        }
#pragma unroll
        for (int kb = 0; kb < kTile / 32; ++kb) {
#pragma unroll
          for (int r = 0; r < 16; ++r) dsb[kb][r] *= __builtin_amdgcn_exp2f(sb[kb][r] * scale_log2 - lse2);
#pragma unroll
          for (int eb = 0; eb < HD / 32; ++eb) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              if constexpr (sizeof(T) == 2) {
                mma16(dqacc[eb], lds_tr_op<T, HD + kPad>(kt, kb, c, eb, lane), pack8<T>(dsb[kb], 8 * c));
              } else {
                const T* row = ktt + tr_row<T, HD>(eb * 32 + col) + kb * 32 + 16 * c;
                mma16(dqacc[eb], load_op_lds_perm<T>(row, half), pack8<T>(dsb[kb], 8 * c));
              }
            }
          }
        }
      } else {
#pragma unroll
        for (int kb = 0; kb < kTile / 32; ++kb) {
          f32x16 s = mask ? bias_init_nb<QUAD, true>(kinfo, knb, tabq, kb, half, qlab)
                          : bias_init_nb<QUAD, false>(kinfo, knb, tabq, kb, half, qlab);
          f32x16 dp;
#pragma unroll
          for (int r = 0; r < 16; ++r) dp[r] = -Dq;      // dP - D straight from the product
#pragma unroll
          for (int c = 0; c < HD / 16; ++c) {
            mma16(s, load_op_lds<T>(kt + (kb * 32 + col) * (HD + kPad) + 16 * c + 8 * half), qop[c]);
            mma16(dp, load_op_lds<T>(vr + (kb * 32 + col) * (HD + kPad) + 16 * c + 8 * half), dop[c]);
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) dsb[kb][r] = __builtin_amdgcn_exp2f(s[r] * scale_log2 - lse2) * dp[r];
#pragma unroll
          for (int eb = 0; eb < HD / 32; ++eb) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              if constexpr (sizeof(T) == 2) {
                mma16(dqacc[eb], lds_tr_op<T, HD + kPad>(kt, kb, c, eb, lane), pack8<T>(dsb[kb], 8 * c));
              } else {
                const T* row = ktt + tr_row<T, HD>(eb * 32 + col) + kb * 32 + 16 * c;
                mma16(dqacc[eb], load_op_lds_perm<T>(row, half), pack8<T>(dsb[kb], 8 * c));
              }
            }
          }
        }
      }
      add_bins(dsb, reinterpret_cast<char*>(dtab + wave * g.nbins + qoff), knb, bf,
               q0 + wave * kWaveQ + kWaveQ <= n && k0 + kTile <= n, half);
    }
    if (qvalid) {
      T* row = dq + wt.tok(g, qi) * g.C + hoff;
#pragma unroll
      for (int eb = 0; eb < HD / 32; ++eb)
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
          const int e = eb * 32 + 8 * grp + 4 * half;
#pragma unroll
          for (int x = 0; x < 4; ++x) row[e + x] = from_float<T>(dqacc[eb][4 * grp + x] * scale);
        }
    }
  }
  lds_barrier();
  float* out = partial + ((int64_t)h * nslice + slice) * g.nbins;
  for (int x = threadIdx.x; x < g.nbins; x += kThreads)
    out[x] = ((dtab[x] + dtab[g.nbins + x]) + dtab[2 * g.nbins + x]) + dtab[3 * g.nbins + x];
}

// ---------------------------------------------------------------------------
// Backward, step 2: dK and dV.  Grid: B * nwin * heads * nkc (key chunks of
// 128; a wave owns 32 keys and walks the window's queries in LDS tiles).
// float32 only: the 16-bit types have a kernel of their own below.
// ---------------------------------------------------------------------------
template <typename T, int HD, bool NHWC, bool QUAD>
__global__ __launch_bounds__(kThreads, 1) void bwd_dkdv_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const T* __restrict__ dout, const float* __restrict__ lse, const float* __restrict__ D,
    const float* __restrict__ table, T* __restrict__ dk, T* __restrict__ dv,
    Geo g, int nkc, float scale_log2, float scale) {
  constexpr int kTile = tile_of<T, HD>();
  extern __shared__ __align__(16) char smem[];
  T* qr = reinterpret_cast<T*>(smem);                 // Q  [kTile][HD+kPad]
  T* dr = qr + kTile * (HD + kPad);                   // dO [kTile][HD+kPad]
  T* qtt = dr + kTile * (HD + kPad);                  // Q^T (transposed tile, fp32)
  T* dtt = qtt + ttile_size<T, HD>();                // dO^T (fp32)
  int* qinfo = reinterpret_cast<int*>(dtt + ttile_size<T, HD>());
  int* qnb = qinfo + kTile;                               // 4 x bias offset per query
  float* ql = reinterpret_cast<float*>(qnb + kTile);     // lse2 per query
  float* qd = ql + kTile;                                 // -D per query
  float* tab = qd + kTile;                                // [nbins+4], forward order
  uint32_t* tt = reinterpret_cast<uint32_t*>(tab + g.nbins + 4);   // [wh*ww] token offsets

  int bid = blockIdx.x;
  const int kc = bid % nkc; bid /= nkc;
  const int h = bid % g.heads; bid /= g.heads;
  const int w = bid % g.nwin;
  const int b = bid / g.nwin;
  const int i = w / g.Mw, j = w - (w / g.Mw) * g.Mw;
  const int cols = win_cols(g, j);
  const int n = win_rows(g, i) * cols;
  const int kbase = kc * kChunk;
  if (kbase >= n) return;
  const WinTokens<NHWC> wt(g, b, i, j);
  const int hoff = h * HD;
  const float bscale = sqrtf((float)HD);
  for (int x = threadIdx.x; x < g.nbins + 4; x += kThreads)
    tab[x] = x < g.nbins ? table[x * g.heads + h] * bscale : -INFINITY;
  const bool mask = window_has_labels(g, i, j) || (n % kTile) != 0;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int ki = kbase + wave * kWaveQ + col;
  const bool kvalid = ki < n;
  const bool wactive = kbase + wave * kWaveQ < n;   // else staging and barriers only
  const int kinf = token_info(g, i, j, cols, kvalid ? ki : 0, n);
  const int klab = kvalid ? (kinf >> 24) : 0xFE;
  const int kfwd = (g.wh - 1) * g.bstride + (g.ww - 1) - (kinf & 0xFFFFFF);
  const char* tabk = reinterpret_cast<const char*>(tab + kfwd);
  const float inv_sl2 = 1.0f / scale_log2;

  typename Operand<T>::type kop[HD / 16], vop[HD / 16];
#pragma unroll
  for (int c = 0; c < HD / 16; ++c) {
    kop[c] = kvalid ? load_op_global<T>(k + wt.tok(g, ki) * g.C + hoff + 16 * c + 8 * half)
                    : zero_op<T>();
    vop[c] = kvalid ? load_op_global<T>(v + wt.tok(g, ki) * g.C + hoff + 16 * c + 8 * half)
                    : zero_op<T>();
  }
  f32x16 dkacc[HD / 32], dvacc[HD / 32];
#pragma unroll
  for (int eb = 0; eb < HD / 32; ++eb) { dkacc[eb] = f32x16{}; dvacc[eb] = f32x16{}; }

  // Q, dO tiles go HBM -> registers -> LDS, one tile ahead up to head dim 64
  constexpr bool kPrefetch = HD <= 64;
  TileRegs<T, HD> rq, rd;
  if (kPrefetch) {
    tile_load(rq, q, g, wt, 0, n, hoff);
    tile_load(rd, dout, g, wt, 0, n, hoff);
  }
  // Head dim 128 (no register prefetch of the tiles): the rows come from
  // the token table, and the per-query words of the next tile are loaded
  // right after the staging barrier so that no wave waits at the barrier for
  // their global loads (backward -7 % at 1024-token windows).  Up to head
  // dim 64 the plain form measured 2 % faster.
  constexpr bool kTab = !kPrefetch;
  if constexpr (kTab) {
    tok_fill(tt, g, wt, n);
    if (NHWC) lds_barrier();   // the first tile comes from the table too
  }
  // Per-query words of a tile (threads below kTile): label/bias word,
  // log-sum-exp in log2 units (+inf for padding queries: P = 0) and -D (the
  // dP accumulator's start).
  int winf = 0;
  float wl = INFINITY, wd = 0.0f;
  auto words = [&](int t0) {
    if (threadIdx.x < kTile) {
      const int t = t0 + threadIdx.x;
      winf = token_info(g, i, j, cols, t, n);
      const int64_t li = t < n ? wt.lse_at(g, h, t) : 0;
      wl = t < n ? lse[li] * kLog2e : INFINITY;
      wd = t < n ? -D[li] : 0.0f;
    }
  };
  if constexpr (kTab) words(0);
  for (int t0 = 0; t0 < n; t0 += kTile) {
    if constexpr (kTab) {
      tile_load_tt(rq, q, g, wt, tt, t0, n, hoff);
      tile_load_tt(rd, dout, g, wt, tt, t0, n, hoff);
    }
    lds_barrier();
    tile_store<T, HD, true, true>(rq, qr, qtt);
    tile_store<T, HD, true, true>(rd, dr, dtt);
    if (threadIdx.x < kTile) {
      if constexpr (kTab) {
        qinfo[threadIdx.x] = winf;
        qnb[threadIdx.x] = 4 * (winf & 0xFFFFFF);
        ql[threadIdx.x] = wl;
        qd[threadIdx.x] = wd;
      } else {
        const int t = t0 + threadIdx.x;
        const int inf = token_info(g, i, j, cols, t, n);
        qinfo[threadIdx.x] = inf;
        qnb[threadIdx.x] = 4 * (inf & 0xFFFFFF);
        const int64_t li = t < n ? wt.lse_at(g, h, t) : 0;
        ql[threadIdx.x] = t < n ? lse[li] * kLog2e : INFINITY;
        qd[threadIdx.x] = t < n ? -D[li] : 0.0f;
      }
    }
    lds_barrier();
    if (t0 + kTile < n) {
      if constexpr (kTab) {
        words(t0 + kTile);
      } else {
        tile_load(rq, q, g, wt, t0 + kTile, n, hoff);
        tile_load(rd, dout, g, wt, t0 + kTile, n, hoff);
      }
    }
    if (!wactive) continue;
    // head_dim 128: one 32-query block at a time (unrolled, the two blocks'
    // operands overlap and the 256 registers spill)
#pragma unroll(HD == 128 ? 1 : kTile / 32)
    for (int qb = 0; qb < kTile / 32; ++qb) {
      // registers 4g..4g+3 hold queries 32qb + 8g + 4*half + 0..3: their
      // log-sum-exp and D are four consecutive LDS words.
      // At head_dim 128 the score accumulator starts at bias - LSE (in
      // score units), as the dP one starts at -D, so that no per-query value
      // stays in registers across the products, and dS replaces dP in place
      // (-20 % spill there; at head_dim 64 the plain form is 1.5 % faster).
      constexpr bool kLean = HD == 128;
      // up to head dim 64, the block's Q and dO operands are read from LDS
      // before its bias (-1 % at 576-token windows)
      constexpr bool kHold = HD <= 64;
      typename Operand<T>::type qo_[kHold ? HD / 16 : 1], do_[kHold ? HD / 16 : 1];
      if constexpr (kHold) {
#pragma unroll
        for (int c = 0; c < HD / 16; ++c) {
          qo_[c] = load_op_lds<T>(qr + (qb * 32 + col) * (HD + kPad) + 16 * c + 8 * half);
          do_[c] = load_op_lds<T>(dr + (qb * 32 + col) * (HD + kPad) + 16 * c + 8 * half);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      // (the byte-offset form costs head dim 128 extra spill)
      f32x16 s;
      if constexpr (HD <= 64)
        s = mask ? bias_init_t_nb<QUAD, true>(qinfo, qnb, tabk, qb, half, klab)
                 : bias_init_t_nb<QUAD, false>(qinfo, qnb, tabk, qb, half, klab);
      else
        s = mask ? bias_init_t<QUAD, true>(qinfo, tab, qb, half, kfwd, klab, g.nbins)
                 : bias_init_t<QUAD, false>(qinfo, tab, qb, half, kfwd, klab, g.nbins);
      f32x16 dp, lq;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4 d4 = *reinterpret_cast<const f32x4*>(qd + qb * 32 + 8 * g4 + 4 * half);
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(ql + qb * 32 + 8 * g4 + 4 * half);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          dp[4 * g4 + x] = d4[x];      // dP - D straight from the product
          if constexpr (kLean) s[4 * g4 + x] -= l4[x] * inv_sl2;
          else lq[4 * g4 + x] = l4[x];
        }
      }
#pragma unroll
      for (int c = 0; c < HD / 16; ++c) {
        if constexpr (kHold) {
          mma16(s, qo_[c], kop[c]);
          mma16(dp, do_[c], vop[c]);
        } else {
          mma16(s, load_op_lds<T>(qr + (qb * 32 + col) * (HD + kPad) + 16 * c + 8 * half), kop[c]);
          mma16(dp, load_op_lds<T>(dr + (qb * 32 + col) * (HD + kPad) + 16 * c + 8 * half), vop[c]);
        }
      }
      f32x16 dsr;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = kLean ? __builtin_amdgcn_exp2f(s[r] * scale_log2)
                              : __builtin_amdgcn_exp2f(s[r] * scale_log2 - lq[r]);
        if constexpr (kLean) dp[r] *= p;          // dS
        else dsr[r] = p * dp[r];
        s[r] = p;
      }
      const f32x16& ds = kLean ? dp : dsr;
#pragma unroll
      for (int eb = 0; eb < HD / 32; ++eb) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int cofs = qb * 32 + 16 * c;
          mma16(dvacc[eb], load_op_lds_perm<T>(dtt + tr_row<T, HD>(eb * 32 + col) + cofs, half),
                pack8<T>(s, 8 * c));
          mma16(dkacc[eb], load_op_lds_perm<T>(qtt + tr_row<T, HD>(eb * 32 + col) + cofs, half),
                pack8<T>(ds, 8 * c));
        }
      }
    }
  }
  if (!kvalid) return;
  T* krow = dk + wt.tok(g, ki) * g.C + hoff;
  T* vrow = dv + wt.tok(g, ki) * g.C + hoff;
#pragma unroll
  for (int eb = 0; eb < HD / 32; ++eb)
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
      const int e = eb * 32 + 8 * grp + 4 * half;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        krow[e + x] = from_float<T>(dkacc[eb][4 * grp + x] * scale);
        vrow[e + x] = from_float<T>(dvacc[eb][4 * grp + x]);
      }
    }
}

// ---------------------------------------------------------------------------
// Forward for the 16-bit types (windows the window-resident kernel does not
// take): fwd_kernel's plan with the staging of bwd_dkdv16_kernel: row
// addresses, bias offsets and labels once per workgroup, K and V through two
// direct-to-LDS buffers, one barrier a tile, O (and O_lo) out in whole row
// pieces, a copy of the walk for masked and unmasked windows.  Bound by vector
// instructions (576 tokens).  Measured (us, before -> now): 144 tokens of 32
// channels 42 -> 34, 576 of 64 with O_lo 1332 -> 1224, 64 of 128 309 -> 218,
// 1024 of 128 with O_lo 1260 -> 1100.
// ---------------------------------------------------------------------------
template <typename T, int HD, bool NHWC, bool QUAD, bool SPLIT, int NW, bool DIRECT = true>
__global__ __launch_bounds__(NW * 64, 2) void fwd16_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const float* __restrict__ table, T* __restrict__ o, T* __restrict__ olo,
    float* __restrict__ lse, Geo g, int nqc, int unit, float scale_log2) {
  constexpr int NT = NW * 64;
  constexpr int kTB = 64 * HD * 2;                    // bytes of one tile
  const int nP = (g.wh * g.ww + 63) & ~63;
  extern __shared__ __align__(16) char smem[];
  char* tiles = smem;                                 // {K, V} x tile_pairs
  uint32_t* tokb = reinterpret_cast<uint32_t*>(smem + tile_pairs(nP) * 2 * kTB);   // [nP] byte offsets
  int* knb = reinterpret_cast<int*>(tokb + nP);       // [nP] 4 x bias offset
  int* klabs = knb + nP;                              // [nP] label
  float* tab = reinterpret_cast<float*>(klabs + nP);  // [nbins+4], reversed

  int bid = xcd_unit_item<false>(blockIdx.x, unit);
  if (bid >= g.B * g.nwin * g.heads * nqc) return;
  const int qc = bid % nqc; bid /= nqc;
  const int h = bid % g.heads; bid /= g.heads;
  const int w = bid % g.nwin;
  const int b = bid / g.nwin;
  const int i = w / g.Mw, j = w - (w / g.Mw) * g.Mw;
  const int cols = win_cols(g, j);
  const int n = win_rows(g, i) * cols;
  const int q0 = qc * NW * 32;
  if (q0 >= n) return;
  const WinTokens<NHWC> wt(g, b, i, j);
  const uint32_t ibytes = (uint32_t)g.HW * (uint32_t)(g.C * 2);
  const int nr = (n + 63) & ~63;
  for (int t = threadIdx.x; t < nr; t += NT) {
    const int inf = token_info(g, i, j, cols, t, n);
    tokb[t] = t < n ? (wt.tok(g, t) - wt.img0) * (uint32_t)(g.C * 2) + (uint32_t)(h * HD * 2) : tile_pad_row<HD>(ibytes);
    knb[t] = 4 * (inf & 0xFFFFFF);
    klabs[t] = inf >> 24;
  }
  const float bscale = sqrtf((float)HD);
  for (int x = threadIdx.x; x < g.nbins + 4; x += NT)
    tab[x] = x < g.nbins ? table[(g.nbins - 1 - x) * g.heads + h] * bscale : -INFINITY;
  const bool mask = window_has_labels(g, i, j) || (n % 64) != 0;

  const int64_t img = (int64_t)wt.img0 * g.C;
  const i32x4 rk = buffer_rsrc(k + img, ibytes), rv = buffer_rsrc(v + img, ibytes);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int qi = q0 + wave * 32 + col;
  const bool qvalid = qi < n;
  const bool wactive = q0 + wave * 32 < n;            // else staging and barriers only
  const int qinf = token_info(g, i, j, cols, qvalid ? qi : 0, n);
  const int qlab = qinf >> 24;
  const char* tabq = reinterpret_cast<const char*>(
      tab + (g.nbins - 1 - ((qinf & 0xFFFFFF) + (g.wh - 1) * g.bstride + (g.ww - 1))));

  lds_barrier();                                      // the row table
  tile_load<HD, NT, DIRECT>(rk, tiles, tokb, 0);
  tile_load<HD, NT, DIRECT>(rv, tiles + kTB, tokb, 0);
  typename Operand<T>::type qop[HD / 16];
  const uint32_t qtok = wt.tok(g, min(qi, n - 1)) * g.C + h * HD;
#pragma unroll
  for (int c = 0; c < HD / 16; ++c)
    qop[c] = qvalid ? load_op_global<T>(q + qtok + 16 * c + 8 * half) : zero_op<T>();
  constexpr float kPOff = __is_same(T, _Float16) ? 7.0f : 0.0f;

  auto walk = [&](auto masked) {
    constexpr bool kMask = decltype(masked)::value;
    TileAddr<HD> ta(lane);
    f32x16 oacc[HD / 32];
#pragma unroll
    for (int eb = 0; eb < HD / 32; ++eb) oacc[eb] = f32x16{};
    float m_run = -1e30f, l_run = 0.0f;               // running max (log2 units) and sum
    int buf = 0;
    for (int t0 = 0; t0 < n; t0 += 64, buf ^= 1) {
      wait_vm<0>();
      lds_barrier();        // tile t0 is in LDS; every wave is done with the other buffer
      if (t0 + 64 < n) {
        tile_load<HD, NT, DIRECT>(rk, tiles + (buf ^ 1) * 2 * kTB, tokb, t0 + 64);
        tile_load<HD, NT, DIRECT>(rv, tiles + (buf ^ 1) * 2 * kTB + kTB, tokb, t0 + 64);
      }
      if (!wactive) continue;
      const char* kt = tiles + buf * 2 * kTB;
      const char* vt = kt + kTB;
      if constexpr (HD == 128) ta.opaque();
      f32x16 s[2];
      float mloc = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        s[kb] = bias_init_lab<QUAD, kMask>(klabs + t0, knb + t0, tabq, kb, half, qlab);
#pragma unroll
        for (int c = 0; c < HD / 16; ++c) mma16(s[kb], tile_row_op<T, HD>(kt, ta, 32 * kb, c), qop[c]);
#pragma unroll
        for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, s[kb][r]);
      }
      mloc = halves_max(mloc);
      // The running maximum moves only past a margin of 2^8: weights below
      // 256 are carried as exactly as weights below 1.  For float16 operands
      // the weights run 2^kPOff higher (m_run sits kPOff below the maximum;
      // the sum, and so the LSE, follow), so that weights down to 2^-21 of
      // the maximum, and the low parts of the split, stay above float16's
      // subnormal range (6.1e-5), which the operands would lose.
      const float mt = mloc * scale_log2;
      if (__builtin_amdgcn_ballot_w64(mt > m_run + (kPOff + 8.0f)) != 0) {
        const float mnew = fmaxf(m_run, mt - kPOff);
        const float alpha = exp2f(m_run - mnew);
        m_run = mnew;
        l_run *= alpha;
#pragma unroll
        for (int eb = 0; eb < HD / 32; ++eb) oacc[eb] *= alpha;
      }
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(s[kb][r] * scale_log2 - m_run);
          s[kb][r] = p;
          l_run += p;
        }
      }
      // With SPLIT, P also enters as hi + lo (lo = P - hi rounded again), so
      // that the fp32 sum carries P V to about 16 significant bits.
      typename Operand<T>::type phi[2][2], plo[2][2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          phi[kb][c] = pack8<T>(s[kb], 8 * c);
          if constexpr (SPLIT) {
#pragma unroll
            for (int x = 0; x < 8; ++x)
              plo[kb][c][x] = from_float<T>(s[kb][8 * c + x] - to_float<T>(phi[kb][c][x]));
          }
        }
#pragma unroll
      for (int eb = 0; eb < HD / 32; ++eb)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const auto vop = tile_tr_op<T, HD>(vt, ta, kb, c, eb);
            mma16(oacc[eb], vop, phi[kb][c]);
            if constexpr (SPLIT) mma16(oacc[eb], vop, plo[kb][c]);
          }
    }
    lds_barrier();
    if (!wactive) return;
    l_run = halves_sum(l_run);
    const float inv = 1.0f / l_run;
    // The split needs one float32 value behind both halves: left to itself
    // the compiler folds the multiply into a float16 mixed-precision multiply
    // on the O_lo side (one rounding of acc * inv) while the stored O rounds
    // the float32 product again, and near a tie the two pick different
    // halves.  OR-ing in a zero the compiler cannot prove (opq) stops that.
    const unsigned opq = (unsigned)g.C >> 31;         // 0: C is positive
    T* et = reinterpret_cast<T*>(tiles) + wave * 32 * HD;
#pragma unroll
    for (int out = 0; out < (SPLIT ? 2 : 1); ++out) {
#pragma unroll
      for (int eb = 0; eb < HD / 32; ++eb)
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
          typedef T v4 __attribute__((ext_vector_type(4)));
          v4 p;
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            float val = oacc[eb][4 * grp + x] * inv;
            if constexpr (SPLIT) val = __uint_as_float(__float_as_uint(val) | opq);
            const T hi = from_float<T>(val);
            p[x] = out == 0 ? hi : from_float<T>(val - to_float<T>(hi));
          }
          *reinterpret_cast<v4*>(et + tile_off<HD>(col, eb * 32 + 8 * grp + 4 * half)) = p;
        }
      __builtin_amdgcn_wave_barrier();
      T* dst = out == 0 ? o : olo;
      constexpr int kCpr = HD / 8;
#pragma unroll
      for (int u = 0; u < kCpr / 2; ++u) {
        const int r = (u * 64 + lane) / kCpr, c = (u * 64 + lane) % kCpr;
        const uint4 x = *reinterpret_cast<const uint4*>(et + tile_off<HD>(r, 8 * c));
        const int t = q0 + wave * 32 + r;
        if (t < n) *reinterpret_cast<uint4*>(reinterpret_cast<char*>(dst + img) + tokb[t] + 16 * c) = x;
      }
      __builtin_amdgcn_wave_barrier();
    }
    if (qvalid && half == 0) lse[wt.lse_at(g, h, qi)] = (m_run + __log2f(l_run)) * kLn2;
  };
  if (mask) walk(std::true_type{});
  else walk(std::false_type{});
}

// ---------------------------------------------------------------------------
// Backward, step 1 for the 16-bit types at 128 channels and long windows:
// bwd_dq_kernel's arithmetic and bins with the staging of bwd_dkdv16_kernel.
// Tiles, bias table and four bin copies leave room for one workgroup a CU,
// and four waves are then one a SIMD.  Here eight waves share the four copies
// in pairs (w, w + 4) by turns: between barriers A and B of a tile the first
// half of the workgroup computes and the second half adds the bins of the
// tile before, between B and the next A they swap, so the order of additions
// stays fixed.  1024 tokens: 2412 -> 1631 us.  (With four waves and two
// workgroups a CU the general kernel is the better one: an item here starts
// with tables of the whole window.  576 tokens of 64 channels 2096 -> 1930 us
// on the 256 x 540 grid, but 0.71 to 0.95x on smaller or odd-width ones.)
// ---------------------------------------------------------------------------
template <typename T, bool NHWC, bool QUAD>
__global__ __launch_bounds__(512, 2) void bwd_dq16_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const T* __restrict__ o, const T* __restrict__ olo,
    const T* __restrict__ dout, const float* __restrict__ lse, float* __restrict__ D,
    const float* __restrict__ table, T* __restrict__ dq, float* __restrict__ partial,
    Geo g, int nqc, int nslice, float scale_log2, float scale) {
  constexpr int HD = 128, NW = 8, NT = NW * 64, kCopies = 4;
  constexpr int kTB = 64 * HD * 2;                    // bytes of one tile
  const int nP = (g.wh * g.ww + 63) & ~63;
  extern __shared__ __align__(16) char smem[];
  char* tiles = smem;                                 // {K, V} x 2 buffers
  uint32_t* tokb = reinterpret_cast<uint32_t*>(smem + 4 * kTB);   // [nP] byte offsets
  float* tab = reinterpret_cast<float*>(tokb + nP);   // [nbins+4], reversed
  float* dtab = tab + g.nbins + 4;                    // [kCopies][nbins]
  uint16_t* knball = reinterpret_cast<uint16_t*>(dtab + kCopies * g.nbins);   // [nP] 4 x bias offset
  uint8_t* klaball = reinterpret_cast<uint8_t*>(knball + nP);                 // [nP] label

  const int bid = xcd_item(blockIdx.x, gridDim.x);
  const int h = bid / nslice;
  const int slice = bid - h * nslice;
  if (h >= g.heads) return;
  const float bscale = sqrtf((float)HD);
  for (int x = threadIdx.x; x < g.nbins + 4; x += NT)
    tab[x] = x < g.nbins ? table[(g.nbins - 1 - x) * g.heads + h] * bscale : -INFINITY;
  for (int x = threadIdx.x; x < kCopies * g.nbins; x += NT) dtab[x] = 0.0f;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, col = lane & 31;
  const bool second = wave >= 4;
  const int nitems = g.B * g.nwin * nqc;
  TileAddr<HD> ta(lane);

  for (int it = slice; it < nitems; it += nslice) {
    const int qc = it % nqc;
    const int w = (it / nqc) % g.nwin;
    const int b = it / (nqc * g.nwin);
    const int i = w / g.Mw, j = w - (w / g.Mw) * g.Mw;
    const int cols = win_cols(g, j);
    const int n = win_rows(g, i) * cols;
    const int q0 = qc * NW * 32;
    if (q0 >= n) continue;
    const WinTokens<NHWC> wt(g, b, i, j);
    const int nt = (n + 63) >> 6;
    const uint32_t ibytes = (uint32_t)g.HW * (uint32_t)(g.C * 2);
    lds_barrier();                    // the previous item is done with the tables and tiles
    for (int t = threadIdx.x; t < 64 * nt; t += NT) {
      const int inf = token_info(g, i, j, cols, t, n);
      tokb[t] =
          t < n ? (wt.tok(g, t) - wt.img0) * (uint32_t)(g.C * 2) + (uint32_t)(h * HD * 2) : tile_pad_row<HD>(ibytes);
      knball[t] = (uint16_t)(4 * (inf & 0xFFFFFF));
      klaball[t] = (uint8_t)(inf >> 24);
    }
    const int64_t img = (int64_t)wt.img0 * g.C;
    const i32x4 rk = buffer_rsrc(k + img, ibytes), rv = buffer_rsrc(v + img, ibytes);
    auto load = [&](int tix, int buf) {
      tile_load<HD, NT, true>(rk, tiles + buf * 2 * kTB, tokb, 64 * tix);
      tile_load<HD, NT, true>(rv, tiles + buf * 2 * kTB + kTB, tokb, 64 * tix);
    };
    const int qi = q0 + wave * 32 + col;
    const bool qvalid = qi < n;
    const bool wactive = q0 + wave * 32 < n;          // else staging and barriers only
    const int qinf = token_info(g, i, j, cols, qvalid ? qi : 0, n);
    const int qlab = (qinf >> 24) & 0xFF;
    const int qoff = (qinf & 0xFFFFFF) + (g.wh - 1) * g.bstride + (g.ww - 1);
    const char* tabq = reinterpret_cast<const char*>(tab + (g.nbins - 1 - qoff));
    const uint32_t qtokn = wt.tok(g, min(qi, n - 1));
    const int64_t lidx = wt.img0 * (uint32_t)g.heads + (uint32_t)(h * g.HW) + (qtokn - wt.img0);
    // +inf for padding queries: their P is exactly 0
    const float lse2 = qvalid ? lse[lidx] * kLog2e : INFINITY;
    const uint32_t qtok = qtokn * g.C + h * HD;
    typename Operand<T>::type qop[HD / 16], dop[HD / 16];
#pragma unroll
    for (int c = 0; c < HD / 16; ++c) {
      qop[c] = qvalid ? load_op_global<T>(q + qtok + 16 * c + 8 * half) : zero_op<T>();
      dop[c] = qvalid ? load_op_global<T>(dout + qtok + 16 * c + 8 * half) : zero_op<T>();
    }
    lds_barrier();                    // the tables
    load(0, 0);
    float dsum = 0.0f;
    const bool sweep = olo == nullptr;
    if (!sweep && qvalid) {
      // D from the forward's output: the two halves of a lane pair hold
      // alternate 8-element runs of the query's row, like dop
#pragma unroll
      for (int c = 0; c < HD / 16; ++c) {
        const auto ov = load_op_global<T>(o + qtok + 16 * c + 8 * half);
        const auto lv = load_op_global<T>(olo + qtok + 16 * c + 8 * half);
#pragma unroll
        for (int x = 0; x < 8; ++x) dsum += to_float<T>(dop[c][x]) * (to_float<T>(ov[x]) + to_float<T>(lv[x]));
      }
    }
    const BinFold bf(g, j, cols, qi, col);

    auto sweeps = [&](auto masked) {
      constexpr bool kMask = decltype(masked)::value;
      auto bias = [&](int t0, int kb) {
        f32x16 c;
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int kk = t0 + 32 * kb + 8 * g4 + 4 * half;
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const int kx = QUAD ? kk : kk + x;
            c[4 * g4 + x] = reinterpret_cast<const float*>(tabq + knball[kx])[QUAD ? x : 0];
            if (kMask && klaball[kx] != qlab) c[4 * g4 + x] = -INFINITY;
          }
        }
        return c;
      };
      int vis = 0;                    // tiles visited by this item; its parity is the buffer
      const int last = (sweep ? 2 : 1) * nt - 1;
      // hands over the tile of visit vis and starts the next visit's load
      auto turn = [&]() {
        wait_vm<0>();
        lds_barrier();
        if (vis < last) load((vis + 1) % nt, (vis + 1) & 1);
      };
      if (sweep) {
        for (int tix = 0; tix < nt; ++tix, ++vis) {
          turn();
          if (!wactive) continue;
          const char* kt = tiles + (vis & 1) * 2 * kTB;
          const char* vr = kt + kTB;
          ta.opaque();
#pragma unroll
          for (int kb = 0; kb < 2; ++kb) {
            f32x16 s = bias(64 * tix, kb);
            f32x16 dp = f32x16{};
#pragma unroll
            for (int c = 0; c < HD / 16; ++c) {
              mma16(s, tile_row_op<T, HD>(kt, ta, 32 * kb, c), qop[c]);
              mma16(dp, tile_row_op<T, HD>(vr, ta, 32 * kb, c), dop[c]);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) dsum += __builtin_amdgcn_exp2f(s[r] * scale_log2 - lse2) * dp[r];
          }
        }
      }
      const float Dq = halves_sum(dsum);
      if (qvalid && half == 0) D[lidx] = Dq;
      // main sweep of the first (kPart 1) or second half of the workgroup,
      // each with its own copy of the code, so that no accumulator is merged
      // between them
      auto main_sweep = [&](auto part) {
        constexpr int kPart = decltype(part)::value;
        f32x16 dqacc[HD / 32];
#pragma unroll
        for (int eb = 0; eb < HD / 32; ++eb) dqacc[eb] = f32x16{};
        f32x16 dsb[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) dsb[kb] = f32x16{};
        auto compute = [&](int tix, int vbuf) {
          const int t0 = 64 * tix;
          const char* kt = tiles + vbuf * 2 * kTB;
          const char* vr = kt + kTB;
          ta.opaque();
#pragma unroll
          for (int kb = 0; kb < 2; ++kb) {
            f32x16 s = bias(t0, kb);
#pragma unroll
            for (int r = 0; r < 16; ++r) dsb[kb][r] = -Dq;      // dP - D straight from the product
#pragma unroll
            for (int c = 0; c < HD / 16; ++c) {
              mma16(s, tile_row_op<T, HD>(kt, ta, 32 * kb, c), qop[c]);
              mma16(dsb[kb], tile_row_op<T, HD>(vr, ta, 32 * kb, c), dop[c]);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) dsb[kb][r] *= __builtin_amdgcn_exp2f(s[r] * scale_log2 - lse2);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              const auto dop_ = pack8<T>(dsb[kb], 8 * c);
#pragma unroll
              for (int eb = 0; eb < HD / 32; ++eb) mma16(dqacc[eb], tile_tr_op<T, HD>(kt, ta, kb, c, eb), dop_);
            }
          }
        };
        auto bins = [&](int t0) {
          add_bins(dsb, reinterpret_cast<char*>(dtab + (wave & 3) * g.nbins + qoff), knball + t0, bf,
                   q0 + wave * kWaveQ + kWaveQ <= n && t0 + 64 <= n, half);
        };
        for (int tix = 0; tix < nt; ++tix, ++vis) {
          turn();                                     // barrier A
          const int buf = vis & 1;
          if constexpr (kPart == 1) {
            if (wactive) compute(tix, buf);
            lds_barrier();                            // barrier B
            if (wactive) bins(64 * tix);
          } else {
            if (wactive && tix > 0) bins(64 * (tix - 1));
            lds_barrier();
            if (wactive) compute(tix, buf);
          }
        }
        lds_barrier();
        if constexpr (kPart == 2)
          if (wactive) bins(64 * (nt - 1));
        if (qvalid) {
          T* row = dq + qtok;
#pragma unroll
          for (int eb = 0; eb < HD / 32; ++eb)
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
              typedef T v4 __attribute__((ext_vector_type(4)));
              v4 p;
#pragma unroll
              for (int x = 0; x < 4; ++x) p[x] = from_float<T>(dqacc[eb][4 * grp + x] * scale);
              *reinterpret_cast<v4*>(row + eb * 32 + 8 * grp + 4 * half) = p;
            }
        }
      };
      if (!second) main_sweep(std::integral_constant<int, 1>{});
      else main_sweep(std::integral_constant<int, 2>{});
    };
    if (window_has_labels(g, i, j) || (n & 63) != 0) sweeps(std::true_type{});
    else sweeps(std::false_type{});
  }
  lds_barrier();
  float* out = partial + ((int64_t)h * nslice + slice) * g.nbins;
  for (int x = threadIdx.x; x < g.nbins; x += NT) {
    float sum = dtab[x];
#pragma unroll
    for (int c = 1; c < kCopies; ++c) sum += dtab[c * g.nbins + x];
    out[x] = sum;
  }
}

// ---------------------------------------------------------------------------
// dK and dV for the 16-bit types.  A workgroup of NW waves owns NW x 32 keys
// of one (window, head) and walks the window's queries in tiles of 64.
// What bounds it: latency, at two waves per SIMD (registers).  So
// * everything per query that does not depend on the tile (row address, bias
//   offset, label, log-sum-exp, D) is worked out once per workgroup into
//   LDS, and direct-to-LDS loads fill two tile buffers (one where the window
//   is a single tile): one barrier a tile, no wait for a load just issued;
// * up to head dim 64 the compiler is held to four phases that each issue
//   the LDS reads of the next;
// * masked and unmasked windows have their own copy of the walk (merged in
//   one loop, the accumulators are copied and spill);
// * all chunks of a window and head go to one XCD, whose L2 then serves
//   their common tiles, and dK, dV leave in whole row pieces.
// Measured (us, before -> now): 64-token windows of 32 channels on 128 x 256
// x 6 heads 28 -> 19, 144 tokens 65 -> 47, 576 tokens of 64 channels 1820 ->
// 1603, 1024 tokens of 128 channels 1650 -> 1381, 64 tokens 458 -> 368.
// ---------------------------------------------------------------------------
template <typename T, int HD, bool NHWC, bool QUAD, int NW, bool DIRECT = true>
__global__ __launch_bounds__(NW * 64, 2) void bwd_dkdv16_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const T* __restrict__ dout, const float* __restrict__ lse, const float* __restrict__ D,
    const float* __restrict__ table, T* __restrict__ dk, T* __restrict__ dv,
    Geo g, int nkc, int unit, float scale_log2, float scale) {
  constexpr int NT = NW * 64;
  constexpr int kTB = 64 * HD * 2;                    // bytes of one tile
  const int nP = (g.wh * g.ww + 63) & ~63;
  extern __shared__ __align__(16) char smem[];
  char* tiles = smem;                                 // {Q, dO} x tile_pairs
  uint32_t* tokb = reinterpret_cast<uint32_t*>(smem + tile_pairs(nP) * 2 * kTB);   // [nP] byte offsets
  int* qnb = reinterpret_cast<int*>(tokb + nP);       // [nP] 4 x bias offset
  int* qlab = qnb + nP;                               // [nP] label
  float* ql = reinterpret_cast<float*>(qlab + nP);     // [nP] log-sum-exp, log2 units
  float* qd = ql + nP;                                // [nP] -D
  float* tab = qd + nP;                               // [nbins+4], forward order

  int bid = xcd_unit_item<true>(blockIdx.x, unit);
  if (bid >= g.B * g.nwin * g.heads * nkc) return;
  const int kc = bid % nkc; bid /= nkc;
  const int h = bid % g.heads; bid /= g.heads;
  const int w = bid % g.nwin;
  const int b = bid / g.nwin;
  const int i = w / g.Mw, j = w - (w / g.Mw) * g.Mw;
  const int cols = win_cols(g, j);
  const int n = win_rows(g, i) * cols;
  const int kbase = kc * NW * 32;
  if (kbase >= n) return;
  const WinTokens<NHWC> wt(g, b, i, j);
  // bias and log-sum-exp in score units (head dim 128) or log2 units
  const float lscale = HD == 128 ? sqrtf((float)HD) : kLog2e;
  const uint32_t ibytes = (uint32_t)g.HW * (uint32_t)(g.C * 2);
  const int nr = (n + 63) & ~63;
  for (int t = threadIdx.x; t < nr; t += NT) {
    const uint32_t tok = wt.tok(g, min(t, n - 1));
    const int inf = token_info(g, i, j, cols, t, n);
    const uint32_t li = wt.img0 * (uint32_t)g.heads + (uint32_t)(h * g.HW) + (tok - wt.img0);
    tokb[t] = t < n ? (tok - wt.img0) * (uint32_t)(g.C * 2) + (uint32_t)(h * HD * 2) : tile_pad_row<HD>(ibytes);
    qnb[t] = 4 * (inf & 0xFFFFFF);
    qlab[t] = inf >> 24;
    ql[t] = t < n ? lse[li] * lscale : INFINITY;      // padding queries: P = 0
    qd[t] = t < n ? -D[li] : 0.0f;
  }
  for (int x = threadIdx.x; x < g.nbins + 4; x += NT)
    tab[x] = x < g.nbins ? table[x * g.heads + h] * lscale : -INFINITY;
  const bool mask = window_has_labels(g, i, j) || (n % 64) != 0;

  const int64_t img = (int64_t)wt.img0 * g.C;
  const i32x4 rq = buffer_rsrc(q + img, ibytes), rd = buffer_rsrc(dout + img, ibytes);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int ki = kbase + wave * 32 + col;
  const bool kvalid = ki < n;
  const bool wactive = kbase + wave * 32 < n;         // else staging and barriers only
  const int kinf = token_info(g, i, j, cols, kvalid ? ki : 0, n);
  const int klab = kvalid ? (kinf >> 24) : 0xFE;
  const int kfwd = (g.wh - 1) * g.bstride + (g.ww - 1) - (kinf & 0xFFFFFF);
  const char* tabk = reinterpret_cast<const char*>(tab + kfwd);

  lds_barrier();                                      // the row table
  tile_load<HD, NT, DIRECT>(rq, tiles, tokb, 0);
  tile_load<HD, NT, DIRECT>(rd, tiles + kTB, tokb, 0);
  typename Operand<T>::type kop[HD / 16], vop[HD / 16];
  const uint32_t ktok = wt.tok(g, min(ki, n - 1)) * g.C + h * HD;
#pragma unroll
  for (int c = 0; c < HD / 16; ++c) {
    kop[c] = kvalid ? load_op_global<T>(k + ktok + 16 * c + 8 * half) : zero_op<T>();
    vop[c] = kvalid ? load_op_global<T>(v + ktok + 16 * c + 8 * half) : zero_op<T>();
  }
  f32x16 dkacc[HD / 32], dvacc[HD / 32];
#pragma unroll
  for (int eb = 0; eb < HD / 32; ++eb) { dkacc[eb] = f32x16{}; dvacc[eb] = f32x16{}; }

  // bias of the block's queries: quads of consecutive queries of one window
  // row where QUAD
  auto bias = [&](int q0, auto masked) {
    f32x16 c;
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int qq = q0 + 8 * g4 + 4 * half;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int qx = QUAD ? qq : qq + x;
        c[4 * g4 + x] = reinterpret_cast<const float*>(tabk + qnb[qx])[QUAD ? x : 0];
        if (decltype(masked)::value && qlab[qx] != klab) c[4 * g4 + x] = -INFINITY;
      }
    }
    return c;
  };
  TileAddr<HD> ta(lane);
  typename Operand<T>::type qop[HD == 128 ? 1 : HD / 16];
  // One block of 32 queries, rows 32 rb of the tile at t0.
  auto body = [&](const char* qr, const char* dr, int t0, int rb, auto masked) {
    const int q0 = t0 + 32 * rb;
    if constexpr (HD == 128) {
      // the score accumulator starts at bias - LSE (score units), the dP one
      // at -D: nothing per query stays in registers across the products
      ta.opaque();
      f32x16 s = bias(q0, masked), dp;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4 d4 = *reinterpret_cast<const f32x4*>(qd + q0 + 8 * g4 + 4 * half);
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(ql + q0 + 8 * g4 + 4 * half);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          dp[4 * g4 + x] = d4[x];
          s[4 * g4 + x] -= l4[x];
        }
      }
#pragma unroll
      for (int c = 0; c < HD / 16; ++c) {
        mma16(s, tile_row_op<T, HD>(qr, ta, 32 * rb, c), kop[c]);
        mma16(dp, tile_row_op<T, HD>(dr, ta, 32 * rb, c), vop[c]);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = __builtin_amdgcn_exp2f(s[r] * scale_log2);
        dp[r] *= s[r];
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const auto pop = pack8<T>(s, 8 * c);
        const auto sop = pack8<T>(dp, 8 * c);
#pragma unroll
        for (int eb = 0; eb < HD / 32; ++eb) {
          mma16(dvacc[eb], tile_tr_op<T, HD>(dr, ta, rb, c, eb), pop);
          mma16(dkacc[eb], tile_tr_op<T, HD>(qr, ta, rb, c, eb), sop);
        }
      }
    } else {
      // Four phases the compiler may not move work across; each issues the
      // LDS reads of the next, so that no product waits for its operands.
      // bias - LSE (log2 units) is added to the scores after the product.
      typename Operand<T>::type dop[HD / 16], dtr[HD / 16], qtr[HD / 16];
      f32x16 s = f32x16{}, dp;
      if (rb == 0) {
#pragma unroll
        for (int c = 0; c < HD / 16; ++c) qop[c] = tile_row_op<T, HD>(qr, ta, 32 * rb, c);
      }
#pragma unroll
      for (int c = 0; c < HD / 16; ++c) dop[c] = tile_row_op<T, HD>(dr, ta, 32 * rb, c);
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4 d4 = *reinterpret_cast<const f32x4*>(qd + q0 + 8 * g4 + 4 * half);
#pragma unroll
        for (int x = 0; x < 4; ++x) dp[4 * g4 + x] = d4[x];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < HD / 16; ++c) mma16(s, qop[c], kop[c]);
      f32x16 bl = bias(q0, masked);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < HD / 16; ++c) mma16(dp, dop[c], vop[c]);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int eb = 0; eb < HD / 32; ++eb) dtr[c * HD / 32 + eb] = tile_tr_op<T, HD>(dr, ta, rb, c, eb);
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(ql + q0 + 8 * g4 + 4 * half);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int r = 4 * g4 + x;
          s[r] = __builtin_amdgcn_exp2f(s[r] * scale_log2 + (bl[r] - l4[x]));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const auto pop = pack8<T>(s, 8 * c);
#pragma unroll
        for (int eb = 0; eb < HD / 32; ++eb) mma16(dvacc[eb], dtr[c * HD / 32 + eb], pop);
      }
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int eb = 0; eb < HD / 32; ++eb) qtr[c * HD / 32 + eb] = tile_tr_op<T, HD>(qr, ta, rb, c, eb);
#pragma unroll
      for (int r = 0; r < 16; ++r) dp[r] *= s[r];
      __builtin_amdgcn_sched_barrier(0);
      if (rb == 0) {
#pragma unroll
        for (int c = 0; c < HD / 16; ++c) qop[c] = tile_row_op<T, HD>(qr, ta, 32, c);
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const auto sop = pack8<T>(dp, 8 * c);
#pragma unroll
        for (int eb = 0; eb < HD / 32; ++eb) mma16(dkacc[eb], qtr[c * HD / 32 + eb], sop);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto tile = [&](const char* qr, const char* dr, int t0, auto masked) {
    if constexpr (HD == 128) {
#pragma unroll 1
      for (int rb = 0; rb < 2; ++rb) body(qr, dr, t0, rb, masked);
    } else {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) body(qr, dr, t0, rb, masked);
    }
  };
  // one copy of the walk for each kind of window: merging the two in the
  // loop costs the accumulators copies and spills
  auto walk = [&](auto masked) {
    int buf = 0;
    for (int t0 = 0; t0 < n; t0 += 64, buf ^= 1) {
      wait_vm<0>();
      lds_barrier();        // tile t0 is in LDS; every wave is done with the other buffer
      if (t0 + 64 < n) {
        tile_load<HD, NT, DIRECT>(rq, tiles + (buf ^ 1) * 2 * kTB, tokb, t0 + 64);
        tile_load<HD, NT, DIRECT>(rd, tiles + (buf ^ 1) * 2 * kTB + kTB, tokb, t0 + 64);
      }
      if (!wactive) continue;
      const char* qr = tiles + buf * 2 * kTB;
      const char* dr = qr + kTB;
      tile(qr, dr, t0, masked);
    }
    // dK, dV rows leave through the wave's own LDS rows (the tile buffers), so
    // that each store instruction moves whole row pieces
    lds_barrier();
    if (!wactive) return;
    T* et = reinterpret_cast<T*>(tiles) + wave * 32 * HD;
  #pragma unroll
    for (int o = 0; o < 2; ++o) {
  #pragma unroll
      for (int eb = 0; eb < HD / 32; ++eb)
  #pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
          typedef T v4 __attribute__((ext_vector_type(4)));
          v4 p;
  #pragma unroll
          for (int x = 0; x < 4; ++x)
            p[x] = from_float<T>(o == 0 ? dkacc[eb][4 * grp + x] * scale : dvacc[eb][4 * grp + x]);
          *reinterpret_cast<v4*>(et + tile_off<HD>(col, eb * 32 + 8 * grp + 4 * half)) = p;
        }
      __builtin_amdgcn_wave_barrier();
      T* dst = o == 0 ? dk : dv;
      constexpr int kCpr = HD / 8;
  #pragma unroll
      for (int u = 0; u < kCpr / 2; ++u) {
        const int r = (u * 64 + lane) / kCpr, c = (u * 64 + lane) % kCpr;
        const uint4 x = *reinterpret_cast<const uint4*>(et + tile_off<HD>(r, 8 * c));
        const int t = kbase + wave * 32 + r;
        if (t < n)
          *reinterpret_cast<uint4*>(reinterpret_cast<char*>(dst + img) + tokb[t] + 16 * c) = x;
      }
      __builtin_amdgcn_wave_barrier();
    }
  };
  if (mask) walk(std::true_type{});
  else walk(std::false_type{});
}

// ---------------------------------------------------------------------------
// Host-side launchers (called by the C ABI after validation).
// ---------------------------------------------------------------------------
static inline int num_chunks(const Geo& g) { return (g.wh * g.ww + kChunk - 1) / kChunk; }

template <typename T, int HD>
static size_t fwd_lds(const Geo& g) {
  constexpr int kTile = tile_of<T, HD>();
  return sizeof(T) * (kTile * (HD + kPad) + tr_size<T, HD>()) + 4 * kTile + 4 * (g.nbins + 4) +
         4 * g.wh * g.ww;
}
// Key tiles the dQ kernel keeps resident for a whole item: every tile of the
// window for 16-bit types, head_dim up to 64 and windows of up to 256 tokens
// (the staging then happens once per item instead of once per tile and
// sweep), else 1 (tiles streamed through one staging buffer).
template <typename T, int HD>
static int dq_tiles(const Geo& g) {
  constexpr int kTile = tile_of<T, HD>();
  if (sizeof(T) != 2 || HD > 64 || g.wh * g.ww > 256) return 1;
  return (g.wh * g.ww + kTile - 1) / kTile;
}
template <typename T, int HD>
static size_t dq_lds(const Geo& g) {
  constexpr int kTile = tile_of<T, HD>();
  const int nt = dq_tiles<T, HD>(g);
  return sizeof(T) * (2 * nt * kTile * (HD + kPad) + ttile_size<T, HD>()) + 8 * nt * kTile +
         4 * (g.nbins + 4) + 16 * g.nbins + 4 * g.wh * g.ww;
}
template <typename T, int HD>
static size_t dkdv_lds(const Geo& g) {
  constexpr int kTile = tile_of<T, HD>();
  return sizeof(T) * (2 * kTile * (HD + kPad) + 2 * ttile_size<T, HD>()) + 16 * kTile + 4 * (g.nbins + 4) +
         (HD > 64 ? 4 * g.wh * g.ww : 0);    // token table (head dim 128 only)
}

// The 16-bit forward: one or two {K, V} tile pairs, three words per window
// token, the bias table.
template <int HD>
static size_t fwd16_lds(const Geo& g) {
  const size_t nP = (g.wh * g.ww + 63) & ~63;
  return tile_pairs((int)nP) * 2 * 64 * HD * 2 + 12 * nP + 4 * (g.nbins + 4);
}
// The 16-bit dQ kernel: two {K, V} tile pairs, seven bytes per window token,
// the bias table and four copies of the bins.
template <int HD>
static size_t dq16_lds(const Geo& g) {
  const size_t nP = (g.wh * g.ww + 63) & ~63;
  return 4 * 64 * HD * 2 + 7 * nP + 4 * (g.nbins + 4) + 16 * g.nbins;
}
// The 16-bit dK/dV kernel: one or two {Q, dO} tile pairs, five words per window
// token, the bias table.
template <int HD>
static size_t dkdv16_lds(const Geo& g) {
  const size_t nP = (g.wh * g.ww + 63) & ~63;
  return tile_pairs((int)nP) * 2 * 64 * HD * 2 + 20 * nP + 4 * (g.nbins + 4);
}

// Per-head slices of the dQ / bias-gradient kernel.  The grid is one round
// of resident workgroups rounded down to whole heads: a grid a few
// workgroups past a round leaves those few to run alone at the end (24 heads
// with ceil(2048 / 24) slices each made 2064 workgroups, 4 rounds and 16
// more).  Measured against 2, 4 and 8 rounds, one was fastest or level on
// every workload.  The launcher asks the runtime how many workgroups one CU
// holds; the workspace (a pure function of the geometry and element type, so
// that it can be queried) is sized for the most the kernel's LDS allows.
constexpr int kF32 = 0, kBF16 = 1;
static int slices_for(const Geo& g, int per_cu) {
  const int items = g.B * g.nwin * num_chunks(g);
  int n = g.cus * per_cu / g.heads;
  if (n > items) n = items;
  return n < 1 ? 1 : n;
}
template <typename T>
static int bwd_nslice_max_t(const Geo& g) {
  const size_t lds = g.hd == 32 ? dq_lds<T, 32>(g) : g.hd == 64 ? dq_lds<T, 64>(g) : dq_lds<T, 128>(g);
  int per_cu = (int)((160 * 1024) / lds);            // four waves a workgroup, at most 32 a CU
  if (per_cu > 8) per_cu = 8;
  return slices_for(g, per_cu < 1 ? 1 : per_cu);
}
#if TERRA_ATTN_T == 0
int bwd_nslice(const Geo& g, int dt) {
  return dt == kF32 ? bwd_nslice_max_t<float>(g) : dt == kBF16 ? bwd_nslice_max_t<__bf16>(g)
                                                               : bwd_nslice_max_t<_Float16>(g);
}
#endif

// True when a slice of the general dQ kernel, per_cu workgroups a CU, holds
// more than 1.2 chunks of a full window: its items in the slice's order, each
// as long as its window has key tiles (the windows of ragged edges count as
// what they are: 21 x 31 windows on 64 x 96 tokens, 3 heads, are 183 chunks of
// at most 256, though 16 full windows a head would be 288).
static bool dq_past_one_round(const Geo& g, int per_cu) {
  constexpr int kMax = 2048;
  const int nqc = num_chunks(g), full = (g.wh * g.ww + 63) / 64;
  const int slices = std::min(kMax, std::max(1, g.cus * per_cu / g.heads));
  if ((int64_t)g.B * (g.H / g.wh) * (g.W / g.ww) * nqc > slices) return true;   // two full chunks in some slice
  int tiles[kMax] = {};
  for (int it = 0; it < g.B * g.nwin * nqc; ++it) {
    const int w = it / nqc % g.nwin, n = win_rows(g, w / g.Mw) * win_cols(g, w % g.Mw);
    if (it % nqc * kChunk >= n) continue;
    if ((tiles[it % slices] += (n + 63) / 64) * 5 > 6 * full) return true;
  }
  return false;
}

// Eight-wave dQ kernel: 128 channels, windows of more than 512 tokens that
// keep at least 7 of 8 waves busy, a plan that fits, and work that the
// general kernel would not do in one round.  Measured against the general
// kernel (whole backward), 256 compute units: where that one has a chunk of
// 128 queries a unit or fewer, it is ahead (1024 tokens 0.91x, 651 tokens
// 0.77 to 0.85x, 768 tokens 0.92x: a chunk of 256 is the longer chain);
// beyond, this one (1024 tokens 1.10 to 1.28x, 651 tokens 1.00 to 1.23x, 768
// tokens 1.12x; 576 tokens, 18 of 24 waves, 0.77x).
static bool dq16_takes(const Geo& g) {
  const int nb = (g.wh * g.ww + 31) / 32, nqc = (nb + 7) / 8;
  return g.hd == 128 && g.wh * g.ww > 512 && 8 * nb >= 7 * 8 * nqc && dq16_lds<128>(g) <= 160 * 1024 &&
         dq_past_one_round(g, (int)((160 * 1024) / dq_lds<__bf16, 128>(g)));
}

// Waves of a 16-bit workgroup whose plan takes `lds` bytes.  Four where two
// workgroups fit a CU's LDS, or where those of four leave no CU a second one
// (1024 tokens of 128 channels, 128 workgroups of four against 64 of eight:
// forward 48 us against 56, backward 147.5 against 150.5; 288 against 144:
// 87 against 58 and 223 against 172), else eight (dK/dV, 1024-token windows of
// 128 channels: 2267 us with four, 1381 with eight).  Windows of up to 256 tokens
// take fewer waves where that leaves fewer of them idle (at 128 channels only
// up to 64 tokens: LDS holds two workgroups a CU whatever their waves; 144
// tokens forward 23 us with two waves, 19 with four); longer ones keep
// four (dK/dV, 576 tokens of 64 channels: 1603 us with four and a half-empty
// last chunk, 1890 with three, 1864 with eight).
template <int HD>
static int waves16(const Geo& g, size_t lds) {
  const int nb = (g.wh * g.ww + 31) / 32;
  int nw = 2 * lds <= 160 * 1024 || g.B * g.nwin * g.heads * ((nb + 3) / 4) <= g.cus ? 4 : 8;
  if (nb <= 8)
    for (int c : {4, 3, 2})
      if (c < nw && (HD == 32 || c != 3) && (HD < 128 || nb <= 2) && (nb + c - 1) / c * c < (nb + nw - 1) / nw * nw) nw = c;
  return nw;
}

// Tensors that the 16-bit kernels may load straight into LDS.  Others (views
// at an odd element of a larger buffer) take one form for all windows: eight
// waves, tiles through registers, pairs one by one.
static bool direct_ok(const void* a, const void* b) { return (((uintptr_t)a | (uintptr_t)b) & 15) == 0; }

template <typename T, int HD, bool NHWC>
static hipError_t fwd_impl(const Geo& g, const void* q, const void* k, const void* v,
                           const float* table, void* o, void* olo, float* lse, hipStream_t st) {
  const float sl2 = kLog2e / sqrtf((float)HD);
  const bool quad = quad_layout(g);
  if constexpr (sizeof(T) == 2) {
    const size_t lds = fwd16_lds<HD>(g);
    const bool direct = direct_ok(k, v);
    const int nw = direct ? waves16<HD>(g, lds) : 8;
    const int nqc = ((g.wh * g.ww + 31) / 32 + nw - 1) / nw;
    const int unit = xcd_unit<HD>(g, nqc);
    const int grid = unit_grid(g.B * g.nwin * g.heads * nqc, unit);
#define TERRA_LAUNCH_FWD(QD, SP, NW_, ...)                                                          \
  hipLaunchKernelGGL((fwd16_kernel<T, HD, NHWC, QD, SP, NW_, ##__VA_ARGS__>), dim3(grid), dim3(NW_ * 64), lds, st,  \
                     (const T*)q, (const T*)k, (const T*)v, table, (T*)o, (T*)olo, lse, g, nqc, unit, sl2)
#define TERRA_LAUNCH_FWDN(NW_)                                \
  do {                                                        \
    if (quad) TERRA_LAUNCH_FWD(true, false, NW_);             \
    else TERRA_LAUNCH_FWD(false, false, NW_);                 \
  } while (0)
    if (!direct) {
      if (olo != nullptr) TERRA_LAUNCH_FWD(false, true, 8, false);
      else TERRA_LAUNCH_FWD(false, false, 8, false);
    } else if (olo != nullptr) {      // windows of more than 256 tokens: four or eight waves
      if (quad && nw == 8) TERRA_LAUNCH_FWD(true, true, 8);
      else if (quad) TERRA_LAUNCH_FWD(true, true, 4);
      else if (nw == 8) TERRA_LAUNCH_FWD(false, true, 8);
      else TERRA_LAUNCH_FWD(false, true, 4);
    } else if (nw == 4) TERRA_LAUNCH_FWDN(4);
    else if (nw == 2) TERRA_LAUNCH_FWDN(2);
    else if (nw == 8) TERRA_LAUNCH_FWDN(8);
    else if constexpr (HD == 32) TERRA_LAUNCH_FWDN(3);
#undef TERRA_LAUNCH_FWDN
#undef TERRA_LAUNCH_FWD
  } else {
    const int nqc = num_chunks(g);
    const int grid = grid8(g.B * g.nwin * g.heads * nqc);
    const size_t lds = fwd_lds<T, HD>(g);
#define TERRA_LAUNCH_FWD(QD)                                                                      \
  hipLaunchKernelGGL((fwd_kernel<T, HD, NHWC, QD>), dim3(grid), dim3(kThreads), lds, st,           \
                     (const T*)q, (const T*)k, (const T*)v, table, (T*)o, lse, g, nqc, sl2)
    if (quad) TERRA_LAUNCH_FWD(true);
    else TERRA_LAUNCH_FWD(false);
#undef TERRA_LAUNCH_FWD
  }
  return hipGetLastError();
}

#if TERRA_ATTN_T == 0
size_t bwd_workspace(const Geo& g, int dt) {
  if (win_bwd_ok(g, dt == 1)) return (size_t)g.heads * win_bwd_nslice(g) * g.nbins * sizeof(float);
  const size_t dbytes = (size_t)g.B * g.heads * g.HW * sizeof(float);
  const size_t pbytes = (size_t)g.heads * bwd_nslice(g, dt) * g.nbins * sizeof(float);
  return ((dbytes + 255) / 256) * 256 + pbytes;
}
#endif

template <typename T, int HD, bool NHWC>
static hipError_t bwd_impl(const Geo& g, const void* q, const void* k, const void* v,
                           const void* o, const void* olo, const void* dout, const float* lse,
                           const float* table, void* dq, void* dk, void* dv, float* dtab,
                           void* ws, hipStream_t st) {
  const size_t dbytes = (size_t)g.B * g.heads * g.HW * sizeof(float);
  float* D = reinterpret_cast<float*>(ws);
  float* partial = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + ((dbytes + 255) / 256) * 256);
  hipError_t e;
  const float sl2 = kLog2e / sqrtf((float)HD);
  const float scale = 1.0f / sqrtf((float)HD);
  const bool quad = quad_layout(g);
  const int nmax = bwd_nslice_max_t<T>(g);
  // one round of resident workgroups, whole heads
  auto slices = [&](const void* fn, int threads, size_t lds, int nqc) {
    int resident = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&resident, fn, threads, lds) != hipSuccess) {
      (void)hipGetLastError();
      resident = 2;
    }
    const int n = std::min(g.B * g.nwin * nqc, g.cus * std::max(resident, 1) / g.heads);
    return std::max(1, std::min(n, nmax));
  };
  int nslice = 1;
  bool dq16 = false;
  if constexpr (sizeof(T) == 2 && HD == 128) {
    const int nqc = (g.wh * g.ww + 255) / 256;
    const size_t lds = dq16_lds<HD>(g);
    dq16 = dq16_takes(g) && direct_ok(k, v);
    if (dq16) {
#define TERRA_LAUNCH_DQ(QD)                                                                          \
  do {                                                                                               \
    nslice = slices(reinterpret_cast<const void*>(&bwd_dq16_kernel<T, NHWC, QD>), 512, lds, nqc);  \
    hipLaunchKernelGGL((bwd_dq16_kernel<T, NHWC, QD>), dim3(grid8(g.heads * nslice)), dim3(512),   \
                       lds, st, (const T*)q, (const T*)k, (const T*)v, (const T*)o, (const T*)olo,     \
                       (const T*)dout, lse, D, table, (T*)dq, partial, g, nqc, nslice, sl2, scale);    \
  } while (0)
      if (quad) TERRA_LAUNCH_DQ(true);
      else TERRA_LAUNCH_DQ(false);
#undef TERRA_LAUNCH_DQ
    }
  }
  if (!dq16) {
    const int nqc = num_chunks(g);
    const size_t lds_dq = dq_lds<T, HD>(g);
#define TERRA_LAUNCH_DQ(QD, RS)                                                                       \
  do {                                                                                                \
    nslice = slices(reinterpret_cast<const void*>(&bwd_dq_kernel<T, HD, NHWC, QD, RS>), kThreads,      \
                    lds_dq, nqc);                                                                     \
    hipLaunchKernelGGL((bwd_dq_kernel<T, HD, NHWC, QD, RS>), dim3(g.heads * nslice), dim3(kThreads),    \
                       lds_dq, st, (const T*)q, (const T*)k, (const T*)v, (const T*)o, (const T*)olo,   \
                       (const T*)dout, lse, D, table, (T*)dq, partial, g, nqc, nslice, sl2, scale);     \
  } while (0)
    const bool res = dq_tiles<T, HD>(g) > 1;
    if constexpr (sizeof(T) == 2 && HD <= 64) {
      if (quad && res) TERRA_LAUNCH_DQ(true, true);
      else if (quad) TERRA_LAUNCH_DQ(true, false);
      else if (res) TERRA_LAUNCH_DQ(false, true);
      else TERRA_LAUNCH_DQ(false, false);
    } else {
      if (quad) TERRA_LAUNCH_DQ(true, false);
      else TERRA_LAUNCH_DQ(false, false);
    }
#undef TERRA_LAUNCH_DQ
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if constexpr (sizeof(T) == 2) {
    const int nb = (g.wh * g.ww + 31) / 32;
    const size_t lds_kv = dkdv16_lds<HD>(g);
    const bool direct = direct_ok(q, dout);
    const int nw = direct ? waves16<HD>(g, lds_kv) : 8;
    const int nkc = (nb + nw - 1) / nw;
    const int unit = xcd_unit<HD>(g, nkc);
    const int grid = unit_grid(g.B * g.nwin * g.heads * nkc, unit);
#define TERRA_LAUNCH_KV(QD, NW_, ...)                                                               \
  hipLaunchKernelGGL((bwd_dkdv16_kernel<T, HD, NHWC, QD, NW_, ##__VA_ARGS__>), dim3(grid), dim3(NW_ * 64), lds_kv, st, \
                     (const T*)q, (const T*)k, (const T*)v, (const T*)dout, lse, D, table,            \
                     (T*)dk, (T*)dv, g, nkc, unit, sl2, scale)
#define TERRA_LAUNCH_KVN(NW_)             \
  do {                                    \
    if (quad) TERRA_LAUNCH_KV(true, NW_); \
    else TERRA_LAUNCH_KV(false, NW_);     \
  } while (0)
    if (!direct) TERRA_LAUNCH_KV(false, 8, false);
    else if (nw == 4) TERRA_LAUNCH_KVN(4);
    else if (nw == 2) TERRA_LAUNCH_KVN(2);
    else if (nw == 8) TERRA_LAUNCH_KVN(8);
    else if constexpr (HD == 32) TERRA_LAUNCH_KVN(3);
#undef TERRA_LAUNCH_KVN
#undef TERRA_LAUNCH_KV
  } else {
    const int nqc = num_chunks(g);
    const int grid = g.B * g.nwin * g.heads * nqc;
    const size_t lds_kv = dkdv_lds<T, HD>(g);
    if (quad)
      hipLaunchKernelGGL((bwd_dkdv_kernel<T, HD, NHWC, true>), dim3(grid), dim3(kThreads), lds_kv, st,
                         (const T*)q, (const T*)k, (const T*)v, (const T*)dout, lse, D, table,
                         (T*)dk, (T*)dv, g, nqc, sl2, scale);
    else
      hipLaunchKernelGGL((bwd_dkdv_kernel<T, HD, NHWC, false>), dim3(grid), dim3(kThreads), lds_kv, st,
                         (const T*)q, (const T*)k, (const T*)v, (const T*)dout, lse, D, table,
                         (T*)dk, (T*)dv, g, nqc, sl2, scale);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_dtab_reduce(g, partial, dtab, nslice, st);
}

// Element type codes of the C ABI: 0 float, 1 bfloat16, 2 float16.

#if TERRA_ATTN_T == 0
// Largest LDS plan of the kernels that a geometry may be given (the eight-wave
// dQ kernel's rule asks for its own plan).
template <typename T, int HD>
static size_t max_lds_hd(const Geo& g) {
  if constexpr (sizeof(T) == 2) return std::max({fwd16_lds<HD>(g), dkdv16_lds<HD>(g), dq_lds<T, HD>(g)});
  else return std::max({fwd_lds<T, HD>(g), dkdv_lds<T, HD>(g), dq_lds<T, HD>(g)});
}
template <typename T>
static size_t max_lds_t(const Geo& g) {
  return g.hd == 32 ? max_lds_hd<T, 32>(g) : g.hd == 64 ? max_lds_hd<T, 64>(g) : max_lds_hd<T, 128>(g);
}

// Waves of a workgroup of the forward (0), dQ (1) or dK/dV (2) kernel for
// tensors that start at a multiple of 16 bytes; 0 where a window-resident
// kernel runs.
template <int HD>
static int waves_of(const Geo& g, int which) {
  return which == 1 ? (dq16_takes(g) ? 8 : 4) : waves16<HD>(g, which == 0 ? fwd16_lds<HD>(g) : dkdv16_lds<HD>(g));
}
int attn_waves(const Geo& g, int dt, int which) {
  if (which == 0 ? win_fwd_ok(g, dt == kBF16) : win_bwd_ok(g, dt == kBF16)) return 0;
  if (dt == kF32) return 4;
  return g.hd == 32 ? waves_of<32>(g, which) : g.hd == 64 ? waves_of<64>(g, which) : waves_of<128>(g, which);
}

size_t attn_max_lds(const Geo& g, int dt) {
  size_t m = dt == kF32 ? max_lds_t<float>(g) : dt == kBF16 ? max_lds_t<__bf16>(g) : max_lds_t<_Float16>(g);
  const bool bf = dt == kBF16;
  if (win_fwd_ok(g, bf) && win_fwd_lds(g) > m) m = win_fwd_lds(g);
  if (win_bwd_ok(g, bf) && win_bwd_lds(g) > m) m = win_bwd_lds(g);
  return m;
}
#endif

template <typename T, bool NHWC>
static hipError_t fwd_generic(const Geo& g, const void* q, const void* k, const void* v,
                              const float* table, void* o, void* olo, float* lse, hipStream_t st) {
  switch (g.hd) {
    case 32: return fwd_impl<T, 32, NHWC>(g, q, k, v, table, o, olo, lse, st);
    case 64: return fwd_impl<T, 64, NHWC>(g, q, k, v, table, o, olo, lse, st);
    default: return fwd_impl<T, 128, NHWC>(g, q, k, v, table, o, olo, lse, st);
  }
}

template <typename T, bool NHWC>
static hipError_t bwd_generic(const Geo& g, const void* q, const void* k, const void* v,
                              const void* o, const void* olo, const void* dout, const float* lse,
                              const float* table, void* dq, void* dk, void* dv, float* dtab, void* ws,
                              hipStream_t st) {
  switch (g.hd) {
    case 32: return bwd_impl<T, 32, NHWC>(g, q, k, v, o, olo, dout, lse, table, dq, dk, dv, dtab, ws, st);
    case 64: return bwd_impl<T, 64, NHWC>(g, q, k, v, o, olo, dout, lse, table, dq, dk, dv, dtab, ws, st);
    default: return bwd_impl<T, 128, NHWC>(g, q, k, v, o, olo, dout, lse, table, dq, dk, dv, dtab, ws, st);
  }
}

// The launchers of one element type (this file is compiled once per type,
// TERRA_ATTN_T = 0 float, 1 bfloat16, 2 float16, so that the kernels build in
// parallel; the type-independent rest belongs to type 0).
#define TERRA_ATTN_FWD(name)                                                                          \
  hipError_t name(const Geo& g, bool nhwc, const void* q, const void* k, const void* v,               \
                  const float* table, void* o, void* olo, float* lse, hipStream_t st)
#define TERRA_ATTN_BWD(name)                                                                          \
  hipError_t name(const Geo& g, bool nhwc, const void* q, const void* k, const void* v, const void* o, \
                  const void* olo, const void* dout, const float* lse, const float* table, void* dq,   \
                  void* dk, void* dv, float* dtab, void* ws, hipStream_t st)
#define TERRA_ATTN_DEFINE(T, fwd, bwd)                                                                \
  TERRA_ATTN_FWD(fwd) {                                                                               \
    return nhwc ? fwd_generic<T, true>(g, q, k, v, table, o, olo, lse, st)                             \
                : fwd_generic<T, false>(g, q, k, v, table, o, olo, lse, st);                           \
  }                                                                                                   \
  TERRA_ATTN_BWD(bwd) {                                                                               \
    return nhwc ? bwd_generic<T, true>(g, q, k, v, o, olo, dout, lse, table, dq, dk, dv, dtab, ws, st)  \
                : bwd_generic<T, false>(g, q, k, v, o, olo, dout, lse, table, dq, dk, dv, dtab, ws, st); \
  }
#if TERRA_ATTN_T == 1
TERRA_ATTN_DEFINE(__bf16, attn_fwd_bf16, attn_bwd_bf16)
#elif TERRA_ATTN_T == 2
TERRA_ATTN_DEFINE(_Float16, attn_fwd_f16, attn_bwd_f16)
#else
TERRA_ATTN_FWD(attn_fwd_bf16);
TERRA_ATTN_BWD(attn_bwd_bf16);
TERRA_ATTN_FWD(attn_fwd_f16);
TERRA_ATTN_BWD(attn_bwd_f16);
TERRA_ATTN_DEFINE(float, attn_fwd_f32, attn_bwd_f32)

// True when the forward writes the rounding residual O_lo and the backward
// takes D from it: 16-bit types on the generic kernels with windows of more
// than 256 tokens.  Smaller windows keep the D sweep, which is cheaper there
// than the split P V product plus the O_lo traffic (measured: 144-token
// windows, hd 32: forward +0.017 ms, backward -0.011 ms; 64-token windows,
// hd 128: forward +0.10 ms, backward +0.10 ms; 576-token windows, hd 64:
// forward +0.26 ms, backward -0.81 ms).
bool attn_uses_olo(const Geo& g, int dt) {
  return dt != kF32 && !win_fwd_ok(g, dt == kBF16) && !win_bwd_ok(g, dt == kBF16) && g.wh * g.ww > 256;
}

// dt: element type code.  nhwc: q, k, v, o (and dout, dq, dk, dv) are
// B x H x W x C read and written in place (the token route fused into the
// kernels), LSE in the same token order; otherwise they are window-major.
// olo (nullable) is written and read only where attn_uses_olo holds.
hipError_t launch_attn_fwd(const Geo& g, int dt, bool nhwc, const void* q, const void* k,
                           const void* v, const float* table, void* o, void* olo, float* lse,
                           hipStream_t st) {
  if (win_fwd_ok(g, dt == kBF16)) return launch_win_fwd(g, nhwc, q, k, v, table, o, lse, st);
  if (!attn_uses_olo(g, dt)) olo = nullptr;
  if (dt == kF32) return attn_fwd_f32(g, nhwc, q, k, v, table, o, nullptr, lse, st);
  if (dt == kBF16) return attn_fwd_bf16(g, nhwc, q, k, v, table, o, olo, lse, st);
  return attn_fwd_f16(g, nhwc, q, k, v, table, o, olo, lse, st);
}

hipError_t launch_attn_bwd(const Geo& g, int dt, bool nhwc, const void* q, const void* k,
                           const void* v, const void* o, const void* olo, const void* dout,
                           const float* lse, const float* table, void* dq, void* dk, void* dv,
                           float* dtab, void* ws, hipStream_t st) {
  if (win_bwd_ok(g, dt == kBF16)) {
    const int nslice = win_bwd_nslice(g);
    float* partial = reinterpret_cast<float*>(ws);
    hipError_t e = launch_win_bwd(g, nhwc, q, k, v, dout, lse, table, dq, dk, dv, partial, nslice, st);
    if (e != hipSuccess) return e;
    return launch_dtab_reduce(g, partial, dtab, nslice, st);
  }
  if (!attn_uses_olo(g, dt)) olo = nullptr;
  if (dt == kF32) return attn_bwd_f32(g, nhwc, q, k, v, o, nullptr, dout, lse, table, dq, dk, dv, dtab, ws, st);
  if (dt == kBF16) return attn_bwd_bf16(g, nhwc, q, k, v, o, olo, dout, lse, table, dq, dk, dv, dtab, ws, st);
  return attn_bwd_f16(g, nhwc, q, k, v, o, olo, dout, lse, table, dq, dk, dv, dtab, ws, st);
}

#endif  // TERRA_ATTN_T

}  // namespace terra
