// Expert FFN of the MoE layer (the expert modules E_e of Algorithm 1) on
// dynamically sized per-expert tensors (Section 4.1), forward and backward.
//
// Every product is one persistent grouped GEMM kernel in "NT" form,
//     C[m, n] = sum_k A[m, k] * B[n, k]     (both operands K-contiguous),
// K tiles of 128 bytes, operand tiles loaded HBM -> LDS by buffer loads,
// double-buffered, with an XOR swizzle that keeps the MFMA fragment reads
// bank-conflict free.
//  * bf16 layers: 4 wavefronts on v_mfma_f32_16x16x32_bf16, two barriers
//    per K step, loads and fragment reads issued one at a time between the
//    MFMAs: on 256x256 tiles (waves of 128x128, one workgroup per CU;
//    ffn_gemm16_kernel) or, for products with few tiles per CU, on tiles of
//    32 to 192 rows and 128 columns (two workgroups per CU;
//    ffn_gemm16_mid_kernel), whose heights the schedule chooses; both add
//    every output's products in the same order.
//  * fp32 layers: v_mfma_f32_32x32x2f32 on tiles of 32 to 192 rows and 128
//    columns, two workgroups per CU (ffn_gemm_f32_kernel).
//  * var-M products (forward H, Y; backward dA, dX): the M dimension of
//    expert e is its row count, read on the device; tiles are listed by a
//    one-workgroup schedule kernel, so no host synchronisation is needed.
//  * var-K products (dW): K of expert e is its row count; the K range is
//    split into chunks only when few experts carry most rows, and split
//    partial sums are added in a fixed order (deterministic).
//  * operands whose contraction index is their row index (the weights in dA
//    and dX, both operands of dW) are read K-major through transposing LDS
//    reads; on large experts dX instead reads a transposed copy of [W1; W3]
//    that the backward writes first.
// The persistent grid maps workgroup b to XCD b % 8 and hands each XCD a
// contiguous run of tiles arranged as 4 M-tiles x 8 N-tiles, so tiles that
// share operand panels share that XCD's L2.
// Epilogues (activation, SwiGLU, activation backward, transposed stores) run
// per wavefront on its fp32 accumulators, staged 16 rows at a time through a
// private LDS strip, and write 16-byte vectors.

#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "ffn.hpp"
#include "sched.hpp"
#include "validate.hpp"

namespace moe {
namespace {

constexpr int kRowBytes = 128;                    // one K tile of one operand row
constexpr int kTileBytes = BM * kRowBytes;        // 32 KB
constexpr int kGroupM = 4;      // M tiles per scheduling group
constexpr int kXcds = 8;
constexpr int64_t kMaxOperandRowBytes = (int64_t(1) << 23) - 64;  // 256 rows < 2^31 bytes
// dx_disp up to this size is produced last in the backward (MI355X has a
// 256 MB last-level cache; measured on a 268 MB dx_disp, T = 32768 tokens of
// d = 2048, k = 2: the dispatch backward reads it in 0.077 ms instead of
// 0.126 ms; on a 1.1 GB one the dX product was 2% slower when run last)
constexpr int64_t kDxLastBytes = int64_t(512) << 20;

enum Act { ACT_RELU = 0, ACT_GELU = 1, ACT_SWIGLU = 2 };

// ---------------------------------------------------------------------------
// activations (shared by forward epilogue, backward epilogue and transposes)
// ---------------------------------------------------------------------------
// The epilogues evaluate these once per output element, so they use the
// hardware base-2 exponential and reciprocal (relative error about 1e-6,
// far below the bf16 rounding of the stored results):
//   e^x = 2^(x log2 e),  sigmoid(h) = 1 / (1 + e^-h),
//   tanh(u) = 1 - 2 / (1 + e^(2u))  (both limits exact: e^(2u) -> inf or 0),
//   and GELU as h sigmoid(2u) (limits: -0 for large negative h, where the
//   exponential overflows to inf, and h for large positive h).
__device__ __forceinline__ float exp_fast(float x) {
  return __builtin_amdgcn_exp2f(x * 1.4426950408889634f);
}
__device__ __forceinline__ float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float tanh_fast(float u) {
  return 1.f - 2.f * rcp_fast(1.f + exp_fast(2.f * u));
}
__device__ __forceinline__ float act_f(float h, int act) {
  if (act == ACT_RELU) return fmaxf(h, 0.f);
  // GELU, tanh form: 0.5 h (1 + tanh(u)) = h sigmoid(2u) = h / (1 + e^(-2u)),
  // u = sqrt(2/pi) (h + 0.044715 h^3); -2u log2(e) = h (c1 + c3 h^2)
  constexpr float c1 = -2.f * 0.7978845608028654f * 1.4426950408889634f;
  constexpr float c3 = c1 * 0.044715f;
  return h * rcp_fast(1.f + __builtin_amdgcn_exp2f(h * __builtin_fmaf(c3, h * h, c1)));
}
__device__ __forceinline__ float act_grad_f(float h, int act) {
  if (act == ACT_RELU) return h > 0.f ? 1.f : 0.f;
  const float u = 0.7978845608028654f * (h + 0.044715f * h * h * h);
  const float th = tanh_fast(u);
  const float du = 0.7978845608028654f * (1.f + 3.f * 0.044715f * h * h);
  return 0.5f * (1.f + th) + 0.5f * h * (1.f - th * th) * du;
}
__device__ __forceinline__ float sigm(float h) { return rcp_fast(1.f + exp_fast(-h)); }

// ---------------------------------------------------------------------------
// schedule
// ---------------------------------------------------------------------------
// Every expert's rows are clamped to its region and to rows_alloc, and the
// tile counts to the host bounds the workspace was sized for, so no later
// kernel can index out of bounds.
__global__ __launch_bounds__(64 * kSchedTasks) void schedule_kernel(
    const int32_t* __restrict__ offsets, const int32_t* __restrict__ rows, const SchedArgs A) {
  const int g = threadIdx.x & 63, E = A.E;
  int m = 0;
  if (g < E) {
    const int64_t off = offsets[g];
    int64_t r = rows[g];
    if (off < 0 || off >= A.rows_alloc) r = 0;
    r = min(r, static_cast<int64_t>(offsets[g + 1]) - off);
    r = min(r, A.rows_alloc - off);
    m = static_cast<int>(max(r, int64_t(0)));
  }
  build_schedule<kSchedTasks>(m, A);
}

// ---------------------------------------------------------------------------
// GEMM core
// ---------------------------------------------------------------------------
// c += a * b over four k values: one 32x32 fp32 block, k = 4 consecutive
// values per lane (one 32-bit element of each of the four words)
__device__ __forceinline__ void mma_f32(floatx16& c, const uint4& a, const uint4& b) {
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
}

// Operand layouts.  Every product is C[m, n] = sum_k A[m, k] B[n, k]; an
// operand is stored either K-contiguous (rows are m (or n), k along each
// row: activations in the forward, weights as out x in) or K-major (rows are
// k, m along each row: the weights in the data-gradient products, and both
// operands of the weight-gradient products, which contract over the
// dispatched rows).
enum Layout { L_KC = 0, L_KM = 1 };

// One operand of one tile (byte pointers, byte strides).
//  KC: base = tile row 0 at k = 0; rows = valid tile rows.
//  KM: base = k-row 0 at tile column 0; rows = valid tile columns; k-rows at
//      or past `split` come from base2 (k counted from split), else base.
//  Gated forward (KC B only): base holds the W1 rows, base2 the W3 rows.
struct Operand {
  const char* base;
  const char* base2;
  int64_t ld;         // bytes between consecutive rows
  int rows;
  int split;
};
struct TileOps {
  Operand a, b;
  int K;              // valid k values; rows / columns / k past the valid ones read as 0
};

// KC LDS tile: row r (0..255) of 128 bytes, its 16-byte chunk c stored at
// r*128 + ((c ^ ((r >> 1) & 7)) << 4).  gfx950 LDS serves 16 lanes of a
// 16-byte access per cycle from 64 banks (256 bytes): the MFMA fragment reads
// touch 16 consecutive rows at one logical chunk; rows alternate bank halves
// and (r >> 1) & 7 spreads each half's 8 rows over its 8 slots.
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }
// KM LDS tile: k-row r of 256 elements, its 32-element segment g stored at
// segment g ^ (r & 3).  A transpose read takes, per 32-lane half, 4
// consecutive k-rows of one 32-element segment (64 bytes of bf16 each); the
// XOR puts those rows in 4 different quarters of the 256-byte bank space.

// Buffer resource over an operand.  Every offset used is below 2^31 (host
// limits; K-major resources are re-based every K step), so 0x80000000 is
// always out of range: a lane given that offset loads zeros, which is how
// ragged rows, columns and K tails are filled.
constexpr uint32_t kOob = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const char* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), static_cast<short>(0),
                                           0x7FFFFFFF, 0x00020000);
}
#define MOE_LDS(p) ((__attribute__((address_space(3))) void*)(p))

typedef short v4s __attribute__((ext_vector_type(4)));
// 4 bf16 of one k-row run, transposed across each 16-lane group (gfx950
// ds_read_b64_tr_b16): lane i = 4a + b of a group gets element b of the run
// addressed by lanes 4r + a, for r = 0..3.
__device__ __forceinline__ uint2 read_tr(const char* p) {
  const v4s v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4s*)(p));
  return __builtin_bit_cast(uint2, v);
}

// ---------------------------------------------------------------------------
// kernel parameters
// ---------------------------------------------------------------------------
enum Mode {
  M_FWD1 = 0,        // H = X W1^T -> A = act(H) [, H saved]
  M_FWD1_SWIGLU = 1, // H1, H3 -> A = silu(H1) H3 [, H1 H3 saved]
  M_STORE = 2,       // plain store (Y, dX)
  M_BWD_DA = 3,      // dA = dY W2 -> dH = dA act'(H)
  M_BWD_DA_SWIGLU = 4,
  M_DW = 5           // var-K weight gradient, fp32
};

struct GemmParams {
  // operands (bytes).  var-M: A rows of the dispatched buffer, B the
  // expert's weights (B2: W3 of the gated forward, or the k-rows from split
  // on of a K-major B).  var-K: A and B dispatched buffers read K-major.
  const char* A; int64_t lda;
  const char* B; const char* B2; int64_t ldb; int64_t b_gstride;
  int K;              // var-M: k values
  int kmsplit;        // var-M, K-major B: first k-row taken from B2
  int N;              // output columns
  int M_out;          // var-K: output rows
  int ntiles;         // tiles along N
  int mtiles_out;     // var-K: tiles along M
  int act;
  // outputs
  char* C; int64_t ldc;           // row-major output (bytes per row)
  char* H1; char* H3; int64_t ldh; // saved / read pre-activations (bytes per row)
  int f;                           // SwiGLU: width of one half
  float* dwA; float* dwB; int64_t dw_gstride; int split_row;
  float* partial; int64_t slot_elems;
  const int32_t* offsets;
  const Sched* sched;
  const int2* mtile;
  const int4* seg;
  int mid_list;       // two-workgroups-per-CU kernels: the tile list
  int dw_h;           // and the units of a weight-gradient tile
};

// Tile order, two levels above each XCD's kGroupM x 8 block of tiles.
// Tiles come in bands of kBandM M-tiles; inside a band, in N-blocks of 8
// columns, and inside an N-block, in M-blocks of kGroupM rows whose tiles
// run M fastest.  The blocks of one N-block follow each other, so the 8
// blocks in flight at once (one per XCD) are 2 N-blocks x 4 M-blocks: 16 x
// 16 tiles that read 16 + 16 operand panels, against 4 + 64 when the XCDs
// take 8 N-blocks of the same 4 M-tiles, and a band's A panels stay in the
// last-level cache while its weight panels stream past.  Partial bands and
// blocks at the edges keep the same order with fewer rows or columns.
constexpr int kBandM = 4 * kGroupM;
__device__ __forceinline__ void decode_banded(int L, int n_mt, int n_nt, int& mt, int& nt) {
  const int full_bands = n_mt / kBandM;
  int r, m0, bh;
  if (L < full_bands * kBandM * n_nt) {
    const int band = L / (kBandM * n_nt);
    r = L - band * kBandM * n_nt;
    m0 = band * kBandM;
    bh = kBandM;
  } else {
    r = L - full_bands * kBandM * n_nt;
    m0 = full_bands * kBandM;
    bh = n_mt - m0;
  }
  const int full_nb = n_nt / 8;
  int n0, w;
  if (r < full_nb * 8 * bh) {
    const int nb = r / (8 * bh);
    r -= nb * 8 * bh;
    n0 = nb * 8;
    w = 8;
  } else {
    r -= full_nb * 8 * bh;
    n0 = full_nb * 8;
    w = n_nt - n0;
  }
  const int full_mb = bh / kGroupM;
  int h;
  if (r < full_mb * kGroupM * w) {
    const int mb = r / (kGroupM * w);
    r -= mb * kGroupM * w;
    m0 += mb * kGroupM;
    h = kGroupM;
  } else {
    r -= full_mb * kGroupM * w;
    m0 += full_mb * kGroupM;
    h = bh - full_mb * kGroupM;
  }
  mt = m0 + r % h;
  nt = n0 + r / h;
}

// The products: PASS names the instance (so each is its own kernel in
// traces) and fixes the operand layouts.
// P_BWD_DX_T is dX with the weights read from a transposed copy,
// K-contiguous like the forward's operands.
enum Pass {
  P_FWD_H = 0, P_FWD_Y = 1, P_BWD_DA = 2, P_BWD_DX = 3, P_BWD_DW2 = 4, P_BWD_DW13 = 5,
  P_BWD_DX_T = 6
};
__host__ __device__ constexpr int a_layout(int pass) {
  return pass == P_BWD_DW2 || pass == P_BWD_DW13 ? L_KM : L_KC;
}
__host__ __device__ constexpr int b_layout(int pass) {
  return pass == P_BWD_DA || pass == P_BWD_DX || pass == P_BWD_DW2 || pass == P_BWD_DW13 ? L_KM
                                                                                          : L_KC;
}

// ---------------------------------------------------------------------------
// bf16 products: four wavefronts of 128x128
// ---------------------------------------------------------------------------
// bf16 layers run every product on 4 wavefronts, one per SIMD, each holding a
// 128x128 block of the 256x256 tile as 64 blocks of 16x16 fp32 accumulators
// (v_mfma_f32_16x16x32_bf16, 256 accumulation registers).  Per K step of 64
// there are two barriers, one after the A and one after the B fragment reads
// of the step's stage.  Between the MFMAs each wave issues, one at a time,
// the fragment reads of the next half step and, once a barrier has freed its
// part of the stage, its share of the direct-to-LDS loads of the step after
// next, so the memory pipeline sees a steady stream of requests while the
// matrix core stays busy.  A 128x128 block reads a third less LDS per MFMA
// than a 128x64 one.
constexpr int kThreads16 = 256;

typedef int intx4 __attribute__((ext_vector_type(4)));

// c += a * b for one 16x16 block.  Lane l = 16 G + c16 supplies row c16 of
// the A and B sub-blocks at k = 8 G .. 8 G + 7 and holds rows 4 G .. 4 G + 3,
// column c16 of the result.  Inline assembly keeps each accumulator in place
// in its accumulation registers through the K loop (compiled MFMAs get their
// accumulators shuffled between loop iterations).  The compiler inserts no
// wait states around it, and none are needed inside the loops:
//  * an accumulator updated again, 64 MFMAs later on 256x256 tiles and 4 RB
//    later on the others (4 at the least), is read as the very registers the
//    earlier MFMA writes, which the hardware forwards without wait states;
//  * an MFMA has read its A and B registers before an LDS read issued after it
//    can return into them (on the smallest tile the next stage's first A
//    fragment is requested right behind the last MFMA that used the registers);
//  * fragments read from LDS are waited for by the compiler, as operands.
// The epilogue waits before it reads the accumulators.
__device__ __forceinline__ void mfma16(floatx4& c, const uint4& a, const uint4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
               : "+a"(c)
               : "v"(__builtin_bit_cast(intx4, a)), "v"(__builtin_bit_cast(intx4, b)));
}

// acc += A_tile * B_tile^T over the whole K extent (see above).  Wave w owns
// tile rows 128 (w >> 1) .. +127 and columns 128 (w & 1) .. +127 (gated
// forward: hidden units 64 (w & 1) .. +63 of W1, then the same units of W3).
// The four stage objects are distinct, and the loop is unrolled by two so
// every LDS access names its object statically: the compiler can then tell
// the loads into one stage from the reads of the other.
template <int ALAY, int BLAY, bool GATED, bool FULL>
__device__ __forceinline__ void mainloop16(const TileOps& op, char* la0, char* lb0, char* la1,
                                           char* lb1, floatx4 (&acc)[8][8], int zt) {
  constexpr int KSTEP = 64;
  const int lane = (static_cast<int>(threadIdx.x) & 63) + zt;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wm = wave >> 1, wn = wave & 1;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int K = op.K;
  const int nk = (K + KSTEP - 1) / KSTEP;
  if (nk <= 0) return;
  const int nk2 = (nk + 1) & ~1;   // odd counts load one all-zero step

  // ---- loads: 1 KB blocks (8 rows of a KC tile: lane l -> row l >> 3,
  // physical chunk l & 7; or 2 k-rows of a KM tile: lane l -> k-row l >> 5,
  // physical elements 8 (l & 31) .. +7); wave w loads blocks 8w .. 8w+7 of
  // A (g = 0..7) and of B (g = 8..15) of every stage.
  const int l3 = lane >> 3;
  const int co0 = ((lane & 7) ^ swz(l3)) * 16, co1 = ((lane & 7) ^ swz(l3 + 8)) * 16;
  const int kr = lane >> 5;            // KM: k-row within the block
  const int pe = (lane & 31) * 8;      // KM: physical element within the k-row
  auto km_col = [&](int q) { return (((pe >> 5) ^ q) << 5) + (pe & 31); };
  const __amdgpu_buffer_rsrc_t ra_t = tile_rsrc(op.a.base);
  const __amdgpu_buffer_rsrc_t rb_t = tile_rsrc(op.b.base);
  const __amdgpu_buffer_rsrc_t rb3_t = tile_rsrc(GATED ? op.b.base2 : op.b.base);
  auto km_rsrc = [&](const Operand& o, int kt, bool second) {
    const int64_t k = static_cast<int64_t>(kt) * KSTEP - (second ? o.split : 0);
    return tile_rsrc((second ? o.base2 : o.base) + k * o.ld);
  };
  // the resources and flags of one K step, set once per step
  struct StepLd {
    __amdgpu_buffer_rsrc_t ra, ra2, rb, rb2;
    int kt;
    bool kfull, kany;
  };
  auto step_ld = [&](int kt) {
    StepLd s;
    s.kt = kt;
    s.kfull = (kt + 1) * KSTEP <= K;
    s.kany = kt * KSTEP < K;
    s.ra = ra_t; s.ra2 = ra_t; s.rb = rb_t; s.rb2 = rb3_t;
    if constexpr (ALAY == L_KM) {
      s.ra = km_rsrc(op.a, kt, false);
      s.ra2 = op.a.base2 ? km_rsrc(op.a, kt, true) : s.ra;
    }
    if constexpr (BLAY == L_KM) {
      s.rb = km_rsrc(op.b, kt, false);
      s.rb2 = op.b.base2 ? km_rsrc(op.b, kt, true) : s.rb;
    }
    return s;
  };
  // block blk of operand o (layout LAY) of step s.kt into dst
  auto load_blk = [&](auto lay, const Operand& o, const __amdgpu_buffer_rsrc_t& rs,
                      const __amdgpu_buffer_rsrc_t& rs2, char* dst, int blk, const StepLd& s,
                      bool gated) {
    constexpr int LAY = decltype(lay)::value;
    const int ld = static_cast<int>(o.ld);
    uint32_t off;
    int soff;
    bool second = false;
    if constexpr (LAY == L_KC) {
      const int co = (blk & 1) ? co1 : co0;
      // gated forward: 64-row groups alternate W1 / W3 rows of 64 hidden units
      const int row0 = gated ? (blk >> 4) * 64 + (blk & 7) * 8 : blk * 8;
      second = gated && ((blk >> 3) & 1);
      off = static_cast<uint32_t>(l3 * ld) + co;
      soff = row0 * ld + s.kt * kRowBytes;
      if (!FULL || !s.kfull) {
        const bool ok = (FULL || row0 + l3 < o.rows) && (s.kfull || s.kt * kRowBytes + co < K * 2);
        if (!ok) off = kOob;
      }
    } else {
      const int krel = 2 * blk;                  // first k-row of the block in the step
      const int kabs = s.kt * KSTEP + krel;
      const int q = (krel + kr) & 3;
      const int col = km_col(q);
      second = kabs >= o.split;
      off = static_cast<uint32_t>(kr * ld + col * 2);
      soff = krel * ld;
      if (!FULL || !s.kfull) {
        const bool ok = (FULL || col < o.rows) && (s.kfull || kabs + kr < K);
        if (!ok) off = kOob;
      }
    }
    if (!s.kany) off = kOob;
    if (second)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs2, MOE_LDS(dst + blk * 1024), 16, off, soff, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, MOE_LDS(dst + blk * 1024), 16, off, soff, 0, 0);
  };
  using KC_ = std::integral_constant<int, L_KC>;
  using KM_ = std::integral_constant<int, L_KM>;
  // one of the wave's 16 loads of a stage
  auto load1 = [&](const StepLd& s, char* sa, char* sb, int g) {
    const int blk = wave * 8 + (g & 7);
    if (g < 8) {
      if constexpr (ALAY == L_KC) load_blk(KC_{}, op.a, s.ra, s.ra2, sa, blk, s, false);
      else load_blk(KM_{}, op.a, s.ra, s.ra2, sa, blk, s, false);
    } else {
      if constexpr (BLAY == L_KC) load_blk(KC_{}, op.b, s.rb, s.rb2, sb, blk, s, GATED);
      else load_blk(KM_{}, op.b, s.rb, s.rb2, sb, blk, s, false);
    }
  };

  // ---- fragments.  KC: lane l = 16 G + c16 reads row c16 of a 16-row block,
  // logical chunk 4h + G (k = 32h + 8G .. +7) of the 128-byte row; the row's
  // swizzle is (c16 >> 1) since blocks start at multiples of 16.
  const int c16 = lane & 15, G = lane >> 4;
  const int fa_kc = (wm * 128 + c16) * kRowBytes, fb_kc = (wn * 128 + c16) * kRowBytes;
  // KM: two transpose reads, k-rows 32h + 8G + (c16 >> 2) and 4 below, columns
  // cb + 4 (c16 & 3) .. +3 (lane 4a + b of a 16-lane group then holds column
  // cb + 4a + b at 4 consecutive k); segment swizzle by k & 3 = c16 >> 2
  auto km_frag = [&](const char* st, int cb, int h) -> uint4 {
    const int phys = (((cb >> 5) ^ (c16 >> 2)) << 5) + (cb & 31) + 4 * (c16 & 3);
    const char* p0 = st + (32 * h + 8 * G + (c16 >> 2)) * 512 + phys * 2;
    const uint2 lo = read_tr(p0);
    const uint2 hi = read_tr(p0 + 4 * 512);
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
  };
  // fragment g of half h: A sub-block g (g < 8) or B sub-block g - 8
  auto read1 = [&](const char* sa, const char* sb, int h, uint4 (&fa)[8], uint4 (&fb)[8], int g) {
    const int sw = ((4 * h + G) ^ (c16 >> 1)) << 4;
    if (g < 8) {
      if constexpr (ALAY == L_KC)
        fa[g] = *reinterpret_cast<const uint4*>(sa + fa_kc + g * 16 * kRowBytes + sw);
      else
        fa[g] = km_frag(sa, wm * 128 + g * 16, h);
    } else {
      if constexpr (BLAY == L_KC)
        fb[g - 8] = *reinterpret_cast<const uint4*>(sb + fb_kc + (g - 8) * 16 * kRowBytes + sw);
      else
        fb[g - 8] = km_frag(sb, wn * 128 + (g - 8) * 16, h);
    }
  };
  uint4 f0a[8], f0b[8], f1a[8], f1b[8];   // fragments of k-half 0 / 1 of a stage

  // Every wave runs the same instruction stream on every tile: rows, columns
  // and K past the valid ones were loaded as zeros, so a wave with no valid
  // rows or columns multiplies zeros, and the epilogue stores none of them.
  // (Skipping such a wave's reads and MFMAs with a branch per group broke
  // the interleaving for the whole tile: a partial tile then took several
  // times as long as a full one.)

  // One K step from stage (ca, cb), the next stage in (na, nb); the loads of
  // step kt + 2 go into (ca, cb): its A part once every wave has read the A
  // fragments of k-half 1, its B part once every wave has read the B ones.
  // Two barriers per step let the 16 loads spread over the last three
  // quarters of the step (one per 6 MFMAs) instead of crowding into the
  // second half.
  auto step = [&](int kt, char* ca, char* cb, const char* na, const char* nb) {
    const StepLd s = step_ld(kt + 2);
    // first quarter: MFMAs 0..31 of k-half 0, reads of the A fragments of k-half 1
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      read1(ca, cb, 1, f1a, f1b, g);
#pragma unroll
      for (int m = 4 * g; m < 4 * g + 4; ++m) mfma16(acc[m >> 3][m & 7], f0a[m >> 3], f0b[m & 7]);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // second quarter: MFMAs 32..63 of k-half 0, reads of the B fragments of
    // k-half 1, the A loads of step kt + 2
#pragma unroll
    for (int g = 8; g < 16; ++g) {
      // A loads 0..5 at groups 8, 9, 11, 12, 14, 15
      if (g % 3 != 1) load1(s, ca, cb, g - 8 - (g - 8) / 3);
      read1(ca, cb, 1, f1a, f1b, g);
#pragma unroll
      for (int m = 4 * g; m < 4 * g + 4; ++m) mfma16(acc[m >> 3][m & 7], f0a[m >> 3], f0b[m & 7]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // stage kt + 1 has landed (only the 6 A loads just issued may be pending)
    __builtin_amdgcn_s_waitcnt(0x0076);   // vmcnt(6) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // second half: MFMAs of k-half 1, reads of the next stage's k-half 0, the
    // B loads of step kt + 2
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      // A loads 6, 7 and the B loads at groups 0, 2, 3, 5, 6, 8, 9, 11, 12, 14
      if (g % 3 != 1 && g < 15) load1(s, ca, cb, 6 + g - (g + 1) / 3);
      read1(na, nb, 0, f0a, f0b, g);
#pragma unroll
      for (int m = 4 * g; m < 4 * g + 4; ++m) mfma16(acc[m >> 3][m & 7], f1a[m >> 3], f1b[m & 7]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  {
    const StepLd s0 = step_ld(0), s1 = step_ld(1);
#pragma unroll
    for (int g = 0; g < 16; ++g) load1(s0, la0, lb0, g);
#pragma unroll
    for (int g = 0; g < 16; ++g) load1(s1, la1, lb1, g);
  }
  __builtin_amdgcn_s_waitcnt(0x4F70);   // vmcnt(16): this wave's stage-0 loads landed
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int g = 0; g < 16; ++g) read1(la0, lb0, 0, f0a, f0b, g);
  for (int kt = 0; kt < nk2; kt += 2) {
    step(kt, la0, lb0, la1, lb1);
    step(kt + 1, la1, lb1, la0, lb0);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);
  __builtin_amdgcn_s_barrier();   // every load landed, every read done: stages are free
  // the epilogue reads the accumulators with ordinary instructions
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
}

// ---------------------------------------------------------------------------
// bf16 products on tiles of 32 to 192 rows, two workgroups per CU
// ---------------------------------------------------------------------------
// The 256x256 kernel holds one wavefront per SIMD (256 accumulation
// registers), so a tile's prologue and epilogue leave the matrix cores idle,
// and its tiles are so large that the last round of them often leaves many
// CUs idle: on short K, few tiles per CU, or an epilogue heavy in VALU work
// that idle time is a large share.  This kernel computes tiles of 128
// columns and RB units of 32 rows (RB = 1 .. 6, per tile) with 4 wavefronts
// of 16 RB x 64 (16 RB accumulation registers, under 256 registers in all)
// and 80 KB of LDS, so two workgroups share each CU and one's epilogue
// overlaps the other's MFMAs.  The heights let the schedule spread an
// expert's rows evenly over just as many tiles as fill whole rounds.  It
// reads more operand bytes per flop than the 256x256 tile, which is why
// large products keep the big tile.  The K loop has the same structure: two
// stages of K 64, two barriers per step, loads and fragment reads issued one
// at a time between the MFMAs.
//
// Wave w owns tile rows 16 RB (w >> 1) .. and columns 64 (w & 1) .. +63
// (gated forward: hidden units 32 (w & 1) .. +31 of W1, then the same units
// of W3).  KC LDS tiles are rows of 128 bytes with the swizzle of the big
// tile; KM tiles are 64 k-rows of 128 elements (256 bytes) with the same XOR
// of 32-element segments by k mod 4 (KM A operands: RB = 4 only).
constexpr int wait_vm_lgkm0(int vm) { return (vm & 15) | ((vm >> 4) << 14) | 0x70; }
constexpr int wait_vm(int vm) { return (vm & 15) | ((vm >> 4) << 14) | 0xF70; }

template <int RB, int ALAY, int BLAY, bool GATED>
__device__ __forceinline__ void mainloop_mid(const TileOps& op, char* la0, char* lb0, char* la1,
                                             char* lb1, floatx4 (&acc)[RB][4], int zt) {
  static_assert(ALAY == L_KC || RB == 4, "K-major A tiles are 128 columns wide");
  constexpr int KSTEP = 64;
  constexpr int KMROW = 256;           // bytes per k-row of a KM tile
  constexpr int NM = 4 * RB;           // MFMAs per k-half: one per accumulator
  static_assert(NM >= 4, "updates of one accumulator are at least 4 MFMAs apart");
  const int lane = (static_cast<int>(threadIdx.x) & 63) + zt;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wm = wave >> 1, wn = wave & 1;
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int K = op.K;
  const int nk = (K + KSTEP - 1) / KSTEP;
  if (nk <= 0) return;
  const int nk2 = (nk + 1) & ~1;   // odd counts load one all-zero step

  // ---- loads: 1 KB blocks (8 rows of a KC tile: lane l -> row l >> 3,
  // physical chunk l & 7; or 4 k-rows of a KM tile: lane l -> k-row l >> 4,
  // physical elements 8 (l & 15) .. +7); of every stage, wave w loads blocks
  // 4i + w of A (i < RB) and of B (i < 4).  A lane's offset within a block
  // has bit 31 set (out of range, reads zeros) where the block's row or
  // column is past the valid ones; past K and past the last step the bit is
  // or-ed in per step.
  const int l3 = lane >> 3;
  const int co = ((lane & 7) ^ swz(l3 + (wave & 1) * 8)) * 16;   // block 4i + w: rows 8(4i + w) + l3
  const int kr = lane >> 4;            // KM: k-row within the block (= k mod 4)
  const int pe = (lane & 15) * 8;      // KM: physical element within the k-row
  const int km_col = (((pe >> 5) ^ kr) << 5) + (pe & 31);
  const __amdgpu_buffer_rsrc_t ra_t = tile_rsrc(op.a.base);
  const __amdgpu_buffer_rsrc_t rb_t = tile_rsrc(op.b.base);
  const __amdgpu_buffer_rsrc_t rb3_t = tile_rsrc(GATED ? op.b.base2 : op.b.base);
  const int lda = static_cast<int>(op.a.ld), ldb = static_cast<int>(op.b.ld);
  auto bad = [](bool b) { return static_cast<uint32_t>(b) << 31; };
  uint32_t offa[ALAY == L_KC ? RB : 1], offb[BLAY == L_KC ? 4 : 1];
  if constexpr (ALAY == L_KC) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
      offa[i] = static_cast<uint32_t>(l3 * lda + co) | bad((4 * i + wave) * 8 + l3 >= op.a.rows);
  } else {
    offa[0] = static_cast<uint32_t>(kr * lda + km_col * 2) | bad(km_col >= op.a.rows);
  }
  // gated: block 4i + w holds rows (hidden units) 32 (i >> 1) + 8w .. +7 of
  // W1 (i even) or W3 (i odd)
  auto brow = [&](int i) { return GATED ? (i >> 1) * 32 + wave * 8 : (4 * i + wave) * 8; };
  if constexpr (BLAY == L_KC) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      offb[i] = static_cast<uint32_t>(l3 * ldb + co) | bad(brow(i) + l3 >= op.b.rows);
  } else {
    offb[0] = static_cast<uint32_t>(kr * ldb + km_col * 2) | bad(km_col >= op.b.rows);
  }
  auto km_rsrc = [&](const Operand& o, int kt, bool second) {
    const int64_t k = static_cast<int64_t>(kt) * KSTEP - (second ? o.split : 0);
    return tile_rsrc((second ? o.base2 : o.base) + k * o.ld);
  };
  // what the loads of one K step share: resources of K-major operands, and
  // for K-contiguous ones the lane's K-tail bit
  struct StepLd {
    __amdgpu_buffer_rsrc_t ra, rb, rb2;
    uint32_t kbad;
    int kt;
  };
  auto step_ld = [&](int kt) {
    StepLd s;
    s.kt = kt;
    s.ra = ra_t; s.rb = rb_t; s.rb2 = rb3_t;
    s.kbad = bad(kt * kRowBytes + co >= K * 2);
    if constexpr (ALAY == L_KM) s.ra = km_rsrc(op.a, kt, false);
    if constexpr (BLAY == L_KM) {
      s.rb = km_rsrc(op.b, kt, false);
      s.rb2 = op.b.base2 ? km_rsrc(op.b, kt, true) : s.rb;
    }
    return s;
  };
  auto issue = [&](const __amdgpu_buffer_rsrc_t& rs, char* dst, uint32_t off, int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, MOE_LDS(dst), 16, off, soff, 0, 0);
  };
  auto load_a = [&](const StepLd& s, char* sa, int i) {
    const int blk = 4 * i + wave;
    if constexpr (ALAY == L_KC)
      issue(s.ra, sa + blk * 1024, offa[i] | s.kbad, blk * 8 * lda + s.kt * kRowBytes);
    else
      issue(s.ra, sa + blk * 1024, offa[0] | bad(s.kt * KSTEP + 4 * blk + kr >= K), 4 * blk * lda);
  };
  auto load_b = [&](const StepLd& s, char* sb, int i) {
    const int blk = 4 * i + wave;
    if constexpr (BLAY == L_KC) {
      if (GATED && (i & 1))
        issue(s.rb2, sb + blk * 1024, offb[i] | s.kbad, brow(i) * ldb + s.kt * kRowBytes);
      else
        issue(s.rb, sb + blk * 1024, offb[i] | s.kbad, brow(i) * ldb + s.kt * kRowBytes);
    } else {
      const int kabs = s.kt * KSTEP + 4 * blk;   // split is a multiple of 8: no block straddles it
      const uint32_t off = offb[0] | bad(kabs + kr >= K);
      if (kabs >= op.b.split) issue(s.rb2, sb + blk * 1024, off, 4 * blk * ldb);
      else issue(s.rb, sb + blk * 1024, off, 4 * blk * ldb);
    }
  };

  // ---- fragments (as in the 256x256 kernel; KM k-rows are 256 bytes)
  const int c16 = lane & 15, G = lane >> 4;
  const int fa_kc = (wm * 16 * RB + c16) * kRowBytes, fb_kc = (wn * 64 + c16) * kRowBytes;
  auto km_frag = [&](const char* st, int cb, int h) -> uint4 {
    const int phys = (((cb >> 5) ^ (c16 >> 2)) << 5) + (cb & 31) + 4 * (c16 & 3);
    const char* p0 = st + (32 * h + 8 * G + (c16 >> 2)) * KMROW + phys * 2;
    const uint2 lo = read_tr(p0);
    const uint2 hi = read_tr(p0 + 4 * KMROW);
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
  };
  auto read_a = [&](const char* sa, int h, uint4 (&fa)[RB], int i) {
    const int sw = ((4 * h + G) ^ (c16 >> 1)) << 4;
    if constexpr (ALAY == L_KC)
      fa[i] = *reinterpret_cast<const uint4*>(sa + fa_kc + i * 16 * kRowBytes + sw);
    else
      fa[i] = km_frag(sa, wm * 64 + i * 16, h);
  };
  auto read_b = [&](const char* sb, int h, uint4 (&fb)[4], int j) {
    const int sw = ((4 * h + G) ^ (c16 >> 1)) << 4;
    if constexpr (BLAY == L_KC)
      fb[j] = *reinterpret_cast<const uint4*>(sb + fb_kc + j * 16 * kRowBytes + sw);
    else
      fb[j] = km_frag(sb, wn * 64 + j * 16, h);
  };
  uint4 f0a[RB], f0b[4], f1a[RB], f1b[4];

  // One K step from stage (ca, cb), the next stage in (na, nb); the loads of
  // step kt + 2 go into (ca, cb).  MFMA m is block (m >> 2, m & 3).  The
  // first quarter reads the A fragments of k-half 1, the second the B
  // fragments and issues the A loads, the second half reads the next stage's
  // k-half 0 and issues the B loads.
  auto step = [&](int kt, char* ca, char* cb, const char* na, const char* nb) {
    const StepLd s = step_ld(kt + 2);
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      read_a(ca, 1, f1a, i);
#pragma unroll
      for (int m = 2 * i; m < 2 * i + 2; ++m) mfma16(acc[m >> 2][m & 3], f0a[m >> 2], f0b[m & 3]);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 2 * RB; ++q) {
      if ((q & 1) == 0) load_a(s, ca, q >> 1);
      // B fragments spread over the quarter (RB = 1: two per MFMA)
#pragma unroll
      for (int j = 4 * q / (2 * RB); j < 4 * (q + 1) / (2 * RB); ++j) read_b(cb, 1, f1b, j);
      const int m = 2 * RB + q;
      mfma16(acc[m >> 2][m & 3], f0a[m >> 2], f0b[m & 3]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // stage kt + 1 has landed (only the RB A loads just issued may be pending)
    __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(RB));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      if (m % RB == 0) load_b(s, cb, m / RB);
#pragma unroll
      for (int r = (RB + 4) * m / NM; r < (RB + 4) * (m + 1) / NM; ++r) {
        if (r < RB) read_a(na, 0, f0a, r);
        else read_b(nb, 0, f0b, r - RB);
      }
      mfma16(acc[m >> 2][m & 3], f1a[m >> 2], f1b[m & 3]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  {
    const StepLd s0 = step_ld(0), s1 = step_ld(1);
#pragma unroll
    for (int i = 0; i < RB; ++i) load_a(s0, la0, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_b(s0, lb0, i);
#pragma unroll
    for (int i = 0; i < RB; ++i) load_a(s1, la1, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_b(s1, lb1, i);
  }
  __builtin_amdgcn_s_waitcnt(wait_vm(RB + 4));   // this wave's stage-0 loads landed
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int i = 0; i < RB; ++i) read_a(la0, 0, f0a, i);
#pragma unroll
  for (int j = 0; j < 4; ++j) read_b(lb0, 0, f0b, j);
  for (int kt = 0; kt < nk2; kt += 2) {
    step(kt, la0, lb0, la1, lb1);
    step(kt + 1, la1, lb1, la0, lb0);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);
  __builtin_amdgcn_s_barrier();   // every load landed, every read done: stages are free
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
}

// A wave's block of RB x CB blocks of 16x16, 2 x 2 waves per workgroup.
template <int RB_, int CB_> struct Tile16 {
  static constexpr int RB = RB_, CB = CB_;
  static constexpr int WR = 16 * RB, WC = 16 * CB;      // wave block
  static constexpr int TM = 2 * WR, TN = 2 * WC;        // workgroup tile
  static constexpr int kP = WC + 4;                     // strip pitch (floats): rows 4 apart
                                                        // fall 16 banks apart
  static constexpr int kStripBytes = 16 * kP * 4;
};
using TileBig = Tile16<8, 8>;
static_assert(TileBig::TM == BM && TileBig::TN == BN, "tile size");
static_assert(2 * TileBig::kStripBytes <= kTileBytes, "two staging strips per operand buffer");
static_assert(2 * Tile16<1, 4>::kStripBytes <= kMidN * kRowBytes, "two staging strips per buffer");
static_assert(Tile16<1, 4>::TN == kMidN && Tile16<1, 4>::TM == kMidUnit, "mid tile size");

// Stage rows 16i .. 16i+15 of the wave's accumulators as fp32, row pitch C::kP.
template <typename C>
__device__ __forceinline__ void stage16(float* strip, const floatx4 (&acc)[C::RB][C::CB], int i,
                                        int lane) {
  const int c16 = lane & 15, G = lane >> 4;
#pragma unroll
  for (int j = 0; j < C::CB; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) strip[(4 * G + q) * C::kP + 16 * j + c16] = acc[i][j][q];
}

// Epilogue of one wave's block (RB x CB blocks of C): 16 accumulator rows at
// a time go through the wave's LDS strip; a lane then finishes 8 consecutive
// columns of a row and writes them as one vector (bf16) or two (fp32 weight
// gradients).  el: the lane index, derived like the strip address from an
// opaque zero the caller produces after its K loop, so nothing the epilogue
// computes per lane is hoisted and held in registers across the K loop.
// empty: a weight-gradient tile with no rows to contract over.
template <int MODE, typename C>
__device__ __forceinline__ void epilogue16(const GemmParams& p,
                                           const floatx4 (&acc)[C::RB][C::CB], float* strip,
                                           int el, int wm, int wn, int g, int slot, int row0,
                                           int m_valid, int n0, bool empty) {
  constexpr int WR = C::WR, WC = C::WC, kP = C::kP;
  using T = uint16_t;
  constexpr int ES = 2;
  const int wr0 = wm * WR;                      // the wave's first tile row
  // weight gradients: where the fp32 result of tile row orow, column gc goes
  // (a split partial-sum slot, or the first or second gradient array)
  auto dw_dst = [&](int orow, int gc) -> float* {
    if (slot >= 0)
      return p.partial + static_cast<int64_t>(slot) * p.slot_elems +
             static_cast<int64_t>(orow) * p.N + gc;
    if (orow < p.split_row)
      return p.dwA + static_cast<int64_t>(g) * p.dw_gstride + static_cast<int64_t>(orow) * p.N + gc;
    return p.dwB + static_cast<int64_t>(g) * p.dw_gstride +
           static_cast<int64_t>(orow - p.split_row) * p.N + gc;
  };
  if constexpr (MODE == M_DW) {
    if (empty) {
      // no rows to contract over (a split expert's last segment may be
      // empty): the tile is zero; each lane stores 8 zeros per row pass straight to memory,
      // with no staging, so the tile costs only its stores.  Every wave
      // of the workgroup takes this path, and none touched the LDS.
      constexpr int LR = WC / 8, RG = 64 / LR;
      const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
      for (int r = 0; r < WR; r += RG) {
        const int lm = wr0 + r + el / LR, gc = n0 + wn * WC + (el % LR) * 8;
        if (lm < m_valid && gc < p.N) {
          float* dst = dw_dst(row0 + lm, gc);
          *reinterpret_cast<float4*>(dst) = zero;
          *reinterpret_cast<float4*>(dst + 4) = zero;
        }
      }
      return;
    }
  }
  // ReLU / GELU layers: the epilogue is specialised on the activation, one
  // uniform branch per tile instead of one per element
  auto epilogue = [&](auto act_c) {
  constexpr int ACT = decltype(act_c)::value;
  if constexpr (MODE == M_FWD1_SWIGLU) {
    // strip columns [0,U): H1, [U,2U): H3 of hidden units n0 + U wn + u, U =
    // WC / 2; LU lanes cover a row's U units, 8 each
    constexpr int U = WC / 2, LU = U / 8, RU = 64 / LU;
#pragma unroll
    for (int i = 0; i < C::RB; ++i) {
      stage16<C>(strip, acc, i, el);
#pragma unroll
      for (int it = 0; it < 16 / RU; ++it) {
        const int r = it * RU + el / LU, u8 = (el % LU) * 8;
        const int lm = wr0 + 16 * i + r;
        const int gc = n0 + wn * U + u8;
        if (lm < m_valid && gc < p.N) {
          // H1 and H3 rounded to bf16 once: the packed bits are stored and
          // their values feed the activation
          float h1[8], h3[8], a[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            h1[e] = strip[r * kP + u8 + e];
            h3[e] = strip[r * kP + U + u8 + e];
          }
          const uint4 b1 = pack8(h1), b3 = pack8(h3);
          unpack8(b1, h1);
          unpack8(b3, h3);
#pragma unroll
          for (int e = 0; e < 8; ++e) a[e] = h1[e] * sigm(h1[e]) * h3[e];
          const int64_t grow = row0 + lm;
          if (p.H1) {
            *reinterpret_cast<uint4*>(p.H1 + grow * p.ldh + static_cast<int64_t>(gc) * ES) = b1;
            *reinterpret_cast<uint4*>(p.H3 + grow * p.ldh + static_cast<int64_t>(gc) * ES) = b3;
          }
          *reinterpret_cast<uint4*>(p.C + grow * p.ldc + static_cast<int64_t>(gc) * ES) = pack8(a);
        }
      }
    }
  } else if constexpr (MODE == M_BWD_DA || MODE == M_BWD_DA_SWIGLU) {
    // dH = dA act'(H): (row block, row group) iterations, each reading 8
    // saved pre-activations (two planes for SwiGLU) per lane, issued kPf
    // iterations ahead of their use into a ring of kPf + 1 registers.  LR
    // lanes cover a row of the wave block, RG rows form a group, GB groups
    // a 16-row block.
    constexpr bool SW = MODE == M_BWD_DA_SWIGLU;
    constexpr int LR = WC / 8, RG = 64 / LR, GB = 16 / RG;
    constexpr int kIt = C::RB * GB, kPf = 4, kRing = kPf + 1;
    uint4 q1[kRing], q3[kRing];
    auto pos = [&](int n, int& lm, int& gc) {
      lm = wr0 + 16 * (n / GB) + RG * (n % GB) + el / LR;
      gc = n0 + wn * WC + (el % LR) * 8;
    };
    auto issue = [&](int n) {
      int lm, gc;
      pos(n, lm, gc);
      const bool ok = lm < m_valid && gc < p.N;
      // out-of-tile lanes read the tile's first valid element instead
      const int64_t o = static_cast<int64_t>(row0 + (ok ? lm : 0)) * p.ldh +
                        static_cast<int64_t>(ok ? gc : n0) * ES;
      q1[n % kRing] = *reinterpret_cast<const uint4*>(p.H1 + o);
      if constexpr (SW) q3[n % kRing] = *reinterpret_cast<const uint4*>(p.H3 + o);
    };
#pragma unroll
    for (int n = 0; n < kPf; ++n) issue(n);
#pragma unroll
    for (int n = 0; n < kIt; ++n) {
      if (n + kPf < kIt) issue(n + kPf);
      if (n % GB == 0) stage16<C>(strip, acc, n / GB, el);
      int lm, gc;
      pos(n, lm, gc);
      if (lm < m_valid && gc < p.N) {
        const int r = RG * (n % GB) + el / LR, c8 = (el % LR) * 8;
        const int64_t grow = row0 + lm;
        float h1[8], g1[8];
        unpack8(q1[n % kRing], h1);
        if constexpr (SW) {
          float h3[8], g3[8];
          unpack8(q3[n % kRing], h3);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            // d silu(h1) h3 / dh1 = h3 sg (1 + h1 (1 - sg)), d / dh3 = h1 sg
            const float da = strip[r * kP + c8 + e];
            const float sg = sigm(h1[e]);
            const float t = da * sg, u = t * h3[e];
            g1[e] = __builtin_fmaf(u, __builtin_fmaf(-h1[e], sg, h1[e]), u);
            g3[e] = t * h1[e];
          }
          *reinterpret_cast<uint4*>(p.C + grow * p.ldc + static_cast<int64_t>(gc) * ES) = pack8(g1);
          *reinterpret_cast<uint4*>(p.C + grow * p.ldc + static_cast<int64_t>(p.f + gc) * ES) = pack8(g3);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            g1[e] = strip[r * kP + c8 + e] * act_grad_f(h1[e], ACT);
          *reinterpret_cast<uint4*>(p.C + grow * p.ldc + static_cast<int64_t>(gc) * ES) = pack8(g1);
        }
      }
    }
  } else {
    constexpr int LR = WC / 8, RG = 64 / LR;   // lanes per row, rows per pass
#pragma unroll
    for (int i = 0; i < C::RB; ++i) {
      stage16<C>(strip, acc, i, el);
#pragma unroll
      for (int it = 0; it < 16 / RG; ++it) {
        const int r = RG * it + el / LR, c8 = (el % LR) * 8;
        const int lm = wr0 + 16 * i + r;
        const int gc = n0 + wn * WC + c8;
        if (lm < m_valid && gc < p.N) {
          const float* sp = strip + r * kP + c8;
          if constexpr (MODE == M_DW) {
            float* dst = dw_dst(row0 + lm, gc);
            *reinterpret_cast<float4*>(dst) = make_float4(sp[0], sp[1], sp[2], sp[3]);
            *reinterpret_cast<float4*>(dst + 4) = make_float4(sp[4], sp[5], sp[6], sp[7]);
          } else {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = sp[e];
            const int64_t grow = row0 + lm;
            if constexpr (MODE == M_FWD1) {
              if constexpr (ACT == ACT_RELU) {
                // ReLU commutes with the rounding to bf16 (round(max(h, 0)) =
                // max(round(h), 0)), and ReLU layers keep A alone
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = fmaxf(v[e], 0.f);
              } else {
                // H rounded to bf16 once: the packed bits are stored and
                // their values feed the activation
                const uint4 hb = pack8(v);
                float hh[8];
                unpack8(hb, hh);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = act_f(hh[e], ACT);
                if (p.H1)
                  *reinterpret_cast<uint4*>(p.H1 + grow * p.ldh + static_cast<int64_t>(gc) * ES) = hb;
              }
            }
            *reinterpret_cast<uint4*>(p.C + grow * p.ldc + static_cast<int64_t>(gc) * ES) = pack8(v);
          }
        }
      }
    }
  }
  };
  if constexpr (MODE == M_FWD1 || MODE == M_BWD_DA) {
    if (p.act == ACT_RELU) epilogue(std::integral_constant<int, ACT_RELU>{});
    else epilogue(std::integral_constant<int, ACT_GELU>{});
  } else {
    epilogue(std::integral_constant<int, ACT_SWIGLU>{});
  }
}

template <int MODE, int PASS>
__global__ __launch_bounds__(kThreads16, 1) void ffn_gemm16_kernel(const GemmParams p) {
  __shared__ __attribute__((aligned(16))) char la0[kTileBytes];
  __shared__ __attribute__((aligned(16))) char lb0[kTileBytes];
  __shared__ __attribute__((aligned(16))) char la1[kTileBytes];
  __shared__ __attribute__((aligned(16))) char lb1[kTileBytes];
  using C = TileBig;
  constexpr int TM = C::TM, TN = C::TN;
  constexpr int ES = 2;
  constexpr bool VARK = MODE == M_DW;
  constexpr bool GATED = MODE == M_FWD1_SWIGLU;
  constexpr int ALAY = a_layout(PASS), BLAY = b_layout(PASS);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const Sched& sc = *p.sched;
  const int n_mt = sc.n_mtiles;
  const int n_items = VARK ? sc.n_segs * p.mtiles_out * p.ntiles : n_mt * p.ntiles;
  const int G = gridDim.x;
  const int lbase = (blockIdx.x % kXcds) * (G / kXcds) + blockIdx.x / kXcds;

  for (int round = 0;; ++round) {
    const int L = round * G + lbase;
    if (L >= n_items) break;
    TileOps op;
    int g, row0, m_valid, n0;
    int slot = -1, mt, nt;
    if constexpr (!VARK) {
      int mti;
      decode_banded(L, n_mt, p.ntiles, mti, nt);
      const int2 tm = p.mtile[mti];
      g = tm.x;
      row0 = p.offsets[g] + tm.y;
      m_valid = min(TM, sc.rows[g] - tm.y);
      op.a = {p.A + static_cast<int64_t>(row0) * p.lda, nullptr, p.lda, m_valid, 0};
      op.K = p.K;
      const char* bg = p.B + static_cast<int64_t>(g) * p.b_gstride;
      if constexpr (GATED) {
        n0 = nt * (TN / 2);
        op.b = {bg + static_cast<int64_t>(n0) * p.ldb,
                p.B2 + static_cast<int64_t>(g) * p.b_gstride + static_cast<int64_t>(n0) * p.ldb,
                p.ldb, min(TN / 2, p.N - n0), 0};
      } else if constexpr (BLAY == L_KC) {
        n0 = nt * TN;
        op.b = {bg + static_cast<int64_t>(n0) * p.ldb, nullptr, p.ldb, min(TN, p.N - n0), 0};
      } else {
        n0 = nt * TN;
        op.b = {bg + static_cast<int64_t>(n0) * ES,
                p.B2 ? p.B2 + static_cast<int64_t>(g) * p.b_gstride + static_cast<int64_t>(n0) * ES
                     : nullptr,
                p.ldb, min(TN, p.N - n0), p.B2 ? p.kmsplit : 0x7FFFFFFF};
      }
    } else {
      const int tmn = p.mtiles_out * p.ntiles;
      const int si = L / tmn;
      decode_banded(L - si * tmn, p.mtiles_out, p.ntiles, mt, nt);
      const int4 sg = p.seg[si];
      g = sg.x;
      slot = sg.w;
      const int k1 = min(sg.z, sc.rows[g]);
      const int64_t krow = static_cast<int64_t>(p.offsets[g]) + sg.y;
      row0 = mt * TM;
      n0 = nt * TN;
      m_valid = min(TM, p.M_out - row0);
      op.a = {p.A + krow * p.lda + static_cast<int64_t>(row0) * ES, nullptr, p.lda, m_valid,
              0x7FFFFFFF};
      op.b = {p.B + krow * p.ldb + static_cast<int64_t>(n0) * ES, nullptr, p.ldb,
              min(TN, p.N - n0), 0x7FFFFFFF};
      op.K = max(0, k1 - sg.y);
    }

    // the main loop derives its per-lane constants from an opaque zero made
    // per tile, so they are recomputed per tile instead of being hoisted out
    // of the tile loop and spilled (their reloads would wait on the loads)
    int zt;
    asm volatile("s_mov_b32 %0, 0" : "=s"(zt));
    floatx4 acc[C::RB][C::CB];
    const bool full = op.a.rows >= TM && op.b.rows >= (GATED ? TN / 2 : TN);
    if (full) mainloop16<ALAY, BLAY, GATED, true>(op, la0, lb0, la1, lb1, acc, zt);
    else mainloop16<ALAY, BLAY, GATED, false>(op, la0, lb0, la1, lb1, acc, zt);

    int z;
    asm volatile("s_mov_b32 %0, 0" : "=s"(z));
    float* strip = reinterpret_cast<float*>((wave < 2 ? la0 : lb0) + (wave & 1) * C::kStripBytes + z);
    epilogue16<MODE, C>(p, acc, strip, lane + z, wm, wn, g, slot, row0, m_valid, n0,
                        VARK && op.K == 0);
    __syncthreads();   // strips are free before the next tile's loads
  }
}

// Item of this workgroup in a round of the two-workgroups-per-CU kernels'
// persistent grid, or -1 when it has none left.  Whole rounds give XCD b % 8 a
// contiguous run of items; the last, partial one is spread over all XCDs the
// same way, on as many workgroups as it has items, so it takes a CU each as
// far as they go.  (The grid follows the most tiles the schedule could list;
// with the runs of a whole round the items of a short one would all fall to
// the first XCDs: 4 experts of 306 rows, K = 2504, N = 1000, 112 tiles on two of
// the eight 44 us, now 29; of 1021 rows, 192 tiles of 192 rows 65 / 38.)
__device__ __forceinline__ int round_item(int round, int n_items) {
  const int b = blockIdx.x, first = round * static_cast<int>(gridDim.x), left = n_items - first;
  const int G = min(static_cast<int>(gridDim.x), (left + kXcds - 1) / kXcds * kXcds);
  if (left <= 0 || b >= G) return -1;
  const int L = first + (b % kXcds) * (G / kXcds) + b / kXcds;
  return L < n_items ? L : -1;
}

// One tile of the two-workgroups-per-CU kernels: var-M tiles of the heights
// the schedule chose, weight-gradient tiles of p.dw_h units of rows.
struct MidTile {
  TileOps op;
  int g, h;                // expert (or its segment's), units of rows
  int row0, m_valid, n0;   // first output row, valid rows, first column
  int slot;                // partial-sum slot, or -1
};

template <int MODE>
__device__ __forceinline__ int mid_items(const GemmParams& p) {
  const Sched& sc = *p.sched;
  return (MODE == M_DW ? sc.n_segs * p.mtiles_out : sc.n_mid[p.mid_list]) * p.ntiles;
}

// Tile L of the launch; ES: bytes per element.
template <int MODE, int PASS, int ES>
__device__ __forceinline__ void mid_operands(const GemmParams& p, int L, MidTile& t) {
  constexpr bool GATED = MODE == M_FWD1_SWIGLU;
  constexpr int BLAY = b_layout(PASS), TN = kMidN;
  const Sched& sc = *p.sched;
  int mt, nt;
  t.slot = -1;
  if constexpr (MODE != M_DW) {
    decode_banded(L, sc.n_mid[p.mid_list], p.ntiles, mt, nt);
    const int2 tm = p.mtile[mt];
    const int g = t.g = tm.x & 255;
    t.h = tm.x >> 8;
    t.row0 = p.offsets[g] + tm.y;
    t.m_valid = min(t.h * kMidUnit, sc.rows[g] - tm.y);
    t.op.a = {p.A + static_cast<int64_t>(t.row0) * p.lda, nullptr, p.lda, t.m_valid, 0};
    t.op.K = p.K;
    const char* bg = p.B + static_cast<int64_t>(g) * p.b_gstride;
    const char* bg2 = p.B2 + static_cast<int64_t>(g) * p.b_gstride;
    t.n0 = nt * (GATED ? TN / 2 : TN);
    if constexpr (GATED) {
      t.op.b = {bg + static_cast<int64_t>(t.n0) * p.ldb, bg2 + static_cast<int64_t>(t.n0) * p.ldb,
                p.ldb, min(TN / 2, p.N - t.n0), 0};
    } else if constexpr (BLAY == L_KC) {
      t.op.b = {bg + static_cast<int64_t>(t.n0) * p.ldb, nullptr, p.ldb, min(TN, p.N - t.n0), 0};
    } else {
      const int64_t o = static_cast<int64_t>(t.n0) * ES;
      t.op.b = {bg + o, p.B2 ? bg2 + o : nullptr, p.ldb, min(TN, p.N - t.n0),
                p.B2 ? p.kmsplit : 0x7FFFFFFF};
    }
  } else {
    const int tmn = p.mtiles_out * p.ntiles;
    const int si = L / tmn;
    decode_banded(L - si * tmn, p.mtiles_out, p.ntiles, mt, nt);
    const int4 sg = p.seg[si];
    t.g = sg.x;
    t.h = p.dw_h;
    t.slot = sg.w;
    const int k1 = min(sg.z, sc.rows[t.g]);
    const int64_t krow = static_cast<int64_t>(p.offsets[t.g]) + sg.y;
    t.row0 = mt * t.h * kMidUnit;
    t.n0 = nt * TN;
    t.m_valid = min(t.h * kMidUnit, p.M_out - t.row0);
    t.op.a = {p.A + krow * p.lda + static_cast<int64_t>(t.row0) * ES, nullptr, p.lda, t.m_valid,
              0x7FFFFFFF};
    t.op.b = {p.B + krow * p.ldb + static_cast<int64_t>(t.n0) * ES, nullptr, p.ldb,
              min(TN, p.N - t.n0), 0x7FFFFFFF};
    t.op.K = max(0, k1 - sg.y);
  }
}

template <int MODE, int PASS>
__global__ __launch_bounds__(kThreads16, 2) void ffn_gemm16_mid_kernel(const GemmParams p) {
  constexpr bool VARK = MODE == M_DW;
  constexpr int kRowsA = (VARK ? kMidDwH : kMidMaxH) * kMidUnit;
  __shared__ __attribute__((aligned(16))) char la0[kRowsA * kRowBytes];
  __shared__ __attribute__((aligned(16))) char lb0[kMidN * kRowBytes];
  __shared__ __attribute__((aligned(16))) char la1[kRowsA * kRowBytes];
  __shared__ __attribute__((aligned(16))) char lb1[kMidN * kRowBytes];
  constexpr bool GATED = MODE == M_FWD1_SWIGLU;
  constexpr int ALAY = a_layout(PASS), BLAY = b_layout(PASS);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int n_items = mid_items<MODE>(p);
  for (int round = 0;; ++round) {
    const int L = round_item(round, n_items);
    if (L < 0) break;
    MidTile t;
    mid_operands<MODE, PASS, 2>(p, L, t);
    auto run = [&](auto hc) {
      constexpr int RB = decltype(hc)::value;
      using C = Tile16<RB, 4>;
      int zt, z;   // opaque zeros: see ffn_gemm16_kernel
      asm volatile("s_mov_b32 %0, 0" : "=s"(zt));
      floatx4 acc[RB][4];
      mainloop_mid<RB, ALAY, BLAY, GATED>(t.op, la0, lb0, la1, lb1, acc, zt);
      asm volatile("s_mov_b32 %0, 0" : "=s"(z));
      float* strip = reinterpret_cast<float*>((wave < 2 ? lb0 : lb1) + (wave & 1) * C::kStripBytes + z);
      epilogue16<MODE, C>(p, acc, strip, lane + z, wm, wn, t.g, t.slot, t.row0, t.m_valid, t.n0,
                          VARK && t.op.K == 0);
    };
    if constexpr (VARK) {
      run(std::integral_constant<int, kMidDwH>{});
    } else {
      switch (t.h) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 4: run(std::integral_constant<int, 4>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        default: run(std::integral_constant<int, 6>{}); break;
      }
    }
    __syncthreads();   // strips are free before the next tile's loads
  }
}

// ---------------------------------------------------------------------------
// fp32 products
// ---------------------------------------------------------------------------
// fp32 matrix cores run at a sixteenth of the bf16 rate, so any tile keeps
// them fed from LDS and the caches; what costs time is tiles that leave
// wavefronts idle.  Every fp32 product therefore runs on tiles of 128 columns
// and RB units of 32 rows, RB chosen per tile by the schedule (weight
// gradients: per product by the host), two workgroups per CU, with
// v_mfma_f32_32x32x2f32.  (8 experts of about 512 rows, d = 256, f = 1024: the
// six products of a step took 991 us on 256x256 tiles and take 249 us; 8 of 4096 rows, 1024 x 4096 SwiGLU: step 25.9 -> 20.8 ms;
// 4 of 64 rows, 64 -> 128 -> 64: 31 -> 13 us against one wavefront per 32x32
// block reading memory directly.)  Wave w of four owns columns 32w .. +31 of the tile
// and all its rows (RB blocks of 32x32); of a gated forward tile (64 hidden
// units of W1 and of W3) units 32 (w & 1) .. +31 of both and row blocks
// w >> 1, (w >> 1) + 2, ..  K steps of 32 go HBM -> LDS by buffer loads, two
// stages, the next step's loads issued before the step's MFMAs.
constexpr int kF32Step = 32;

// LDS tiles.  K-contiguous: rows of 128 bytes with the swizzle of the bf16
// tiles.  K-major: 32 k-rows of SEG segments of 32 elements (SEG = RB for A,
// 4 for B), segment s of k-row k stored at s ^ (k & (SEG - 1)).
template <int NB> struct AccF32 { floatx16 v[NB]; };   // row blocks of a wave

template <int RB, int PASS, bool GATED, int NB>
__device__ __forceinline__ void mainloop_f32(const TileOps& op, char* la0, char* lb0, char* la1,
                                             char* lb1, AccF32<NB>& acc_, AccF32<NB>& acc3_) {
  static_assert(NB == (GATED ? (RB + 1) / 2 : RB), "row blocks per wave");
  constexpr int ALAY = a_layout(PASS), BLAY = b_layout(PASS);
  floatx16(&acc)[NB] = acc_.v;
  floatx16(&acc3)[NB] = acc3_.v;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      acc[i][q] = 0.f;
      if constexpr (GATED) acc3[i][q] = 0.f;
    }
  const int K = op.K;
  const int nk = (K + kF32Step - 1) / kF32Step;
  if (nk <= 0) return;
  // ---- loads: 1 KB blocks 4i + w of A (i < RB) and of B (i < 4)
  const int l3 = lane >> 3;
  const int co = ((lane & 7) ^ swz(l3 + (wave & 1) * 8)) * 16;   // KC: block rows 8(4i + w) + l3
  const int lda = static_cast<int>(op.a.ld), ldb = static_cast<int>(op.b.ld);
  auto bad = [](bool b) { return static_cast<uint32_t>(b) << 31; };
  // KM: a block is 8 / SEG k-rows of SEG segments; the lane's k-row within
  // it and physical element
  auto km_row = [&](int seg) { return lane / (8 * seg); };
  auto km_elem = [&](int seg) { return (lane % (8 * seg)) * 4; };
  auto brow = [&](int i) { return GATED ? (i >> 1) * 32 + wave * 8 : (4 * i + wave) * 8; };
  const __amdgpu_buffer_rsrc_t ra_t = tile_rsrc(op.a.base);
  const __amdgpu_buffer_rsrc_t rb_t = tile_rsrc(op.b.base);
  const __amdgpu_buffer_rsrc_t rb3_t = tile_rsrc(GATED ? op.b.base2 : op.b.base);
  auto load_km = [&](auto seg_c, const Operand& o, char* dst, int i, int kt, int ld) {
    constexpr int SEG = decltype(seg_c)::value;
    const int blk = 4 * i + wave;
    const int k0 = blk * (8 / SEG), kr = km_row(SEG);      // first k-row of the block, the lane's
    const int pe = km_elem(SEG);
    const int col = (((pe >> 5) ^ ((k0 + kr) & (SEG - 1))) << 5) + (pe & 31);
    const int kabs = kt * kF32Step + k0;
    const bool second = kabs >= o.split;                   // a multiple of 8
    const int64_t kb = static_cast<int64_t>(kt) * kF32Step - (second ? o.split : 0);
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc((second ? o.base2 : o.base) + kb * o.ld);
    const uint32_t off = static_cast<uint32_t>(kr * ld + col * 4) | bad(col >= o.rows || kabs + kr >= K);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, MOE_LDS(dst + blk * 1024), 16, off, k0 * ld, 0, 0);
  };
  auto load = [&](int kt, char* sa, char* sb) {
    const uint32_t kbad = bad(kt * kRowBytes + co >= K * 4);
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      if constexpr (ALAY == L_KC) {
        const int blk = 4 * i + wave;
        const uint32_t off = static_cast<uint32_t>(l3 * lda + co) | bad(blk * 8 + l3 >= op.a.rows) | kbad;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra_t, MOE_LDS(sa + blk * 1024), 16, off,
                                                 blk * 8 * lda + kt * kRowBytes, 0, 0);
      } else {
        load_km(std::integral_constant<int, RB>{}, op.a, sa, i, kt, lda);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (BLAY == L_KC) {
        const int blk = 4 * i + wave;
        const uint32_t off = static_cast<uint32_t>(l3 * ldb + co) | bad(brow(i) + l3 >= op.b.rows) | kbad;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(GATED && (i & 1) ? rb3_t : rb_t,
                                                 MOE_LDS(sb + blk * 1024), 16, off,
                                                 brow(i) * ldb + kt * kRowBytes, 0, 0);
      } else {
        load_km(std::integral_constant<int, 4>{}, op.b, sb, i, kt, ldb);
      }
    }
  };
  // ---- fragments.  MFMA operand of lane l: row/column l % 32 of the block,
  // k values 8 s + 4 (l / 32) .. +3 of sub-step s
  const int r32 = lane & 31, kh = lane >> 5;
  auto frag_kc = [&](const char* st, int blk, int s) {
    const int row = blk * 32 + r32;
    return *reinterpret_cast<const uint4*>(st + row * kRowBytes + (((2 * s + kh) ^ swz(row)) << 4));
  };
  auto frag_km = [&](auto seg_c, const char* st, int blk, int s) {
    constexpr int SEG = decltype(seg_c)::value;
    uint32_t v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int k = 8 * s + 4 * kh + c;
      v[c] = *reinterpret_cast<const uint32_t*>(
          st + (k * SEG + (blk ^ (c & (SEG - 1)))) * 128 + r32 * 4);   // k & (SEG - 1) = c & (SEG - 1)
    }
    return make_uint4(v[0], v[1], v[2], v[3]);
  };
  auto compute = [&](const char* sa, const char* sb) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      uint4 b, b3;
      if constexpr (GATED) {
        b = frag_kc(sb, 2 * (wave & 1), s);
        b3 = frag_kc(sb, 2 * (wave & 1) + 1, s);
      } else if constexpr (BLAY == L_KC) {
        b = frag_kc(sb, wave, s);
      } else {
        b = frag_km(std::integral_constant<int, 4>{}, sb, wave, s);
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int blk = GATED ? min(2 * i + (wave >> 1), RB - 1) : i;
        uint4 a;
        if constexpr (ALAY == L_KC) a = frag_kc(sa, blk, s);
        else a = frag_km(std::integral_constant<int, RB>{}, sa, blk, s);
        mma_f32(acc[i], a, b);
        if constexpr (GATED) mma_f32(acc3[i], a, b3);
      }
    }
  };
  load(0, la0, lb0);
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  __builtin_amdgcn_s_barrier();
  auto step = [&](int kt, char* ca, char* cb, char* na, char* nb) {
    if (kt + 1 < nk) load(kt + 1, na, nb);
    __builtin_amdgcn_sched_barrier(0);
    compute(ca, cb);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };
  for (int kt = 0; kt < nk; kt += 2) {
    step(kt, la0, lb0, la1, lb1);
    if (kt + 1 < nk) step(kt + 1, la1, lb1, la0, lb0);
  }
}

template <int MODE, int PASS>
__global__ __launch_bounds__(kThreads16, 2) void ffn_gemm_f32_kernel(const GemmParams p) {
  constexpr bool VARK = MODE == M_DW;
  constexpr int kRowsA = (VARK ? 4 : kMidMaxH) * kMidUnit;
  __shared__ __attribute__((aligned(16))) char la0[kRowsA * kRowBytes];
  __shared__ __attribute__((aligned(16))) char lb0[kMidN * kRowBytes];
  __shared__ __attribute__((aligned(16))) char la1[kRowsA * kRowBytes];
  __shared__ __attribute__((aligned(16))) char lb1[kMidN * kRowBytes];
  constexpr bool GATED = MODE == M_FWD1_SWIGLU;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int n_items = mid_items<MODE>(p);
  for (int round = 0;; ++round) {
    const int L = round_item(round, n_items);
    if (L < 0) break;
    MidTile t;
    mid_operands<MODE, PASS, 4>(p, L, t);
    auto run = [&](auto hc) {
      constexpr int RB = decltype(hc)::value;
      constexpr int NB = GATED ? (RB + 1) / 2 : RB;
      AccF32<NB> c1, c3;   // c3: the W3 half of a gated tile
      mainloop_f32<RB, PASS, GATED, NB>(t.op, la0, lb0, la1, lb1, c1, c3);
      floatx16(&acc)[NB] = c1.v;
      floatx16(&acc3)[NB] = c3.v;
      // accumulator q of lane l: column l % 32, row 8 (q / 4) + 4 (l / 32) + q % 4
      const int col = t.n0 + (GATED ? wave & 1 : wave) * 32 + (lane & 31);
      if (col >= p.N) return;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int blk = GATED ? 2 * i + (wave >> 1) : i;
        if (GATED && blk >= RB) continue;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int lm = blk * 32 + 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3);
          if (lm >= t.m_valid) continue;
          const int64_t row = t.row0 + lm;
          if constexpr (MODE == M_DW) {
            float* dst;
            if (t.slot >= 0) dst = p.partial + static_cast<int64_t>(t.slot) * p.slot_elems + row * p.N;
            else if (row < p.split_row) dst = p.dwA + static_cast<int64_t>(t.g) * p.dw_gstride + row * p.N;
            else dst = p.dwB + static_cast<int64_t>(t.g) * p.dw_gstride + (row - p.split_row) * p.N;
            dst[col] = acc[i][q];
          } else {
            float* c = reinterpret_cast<float*>(p.C + row * p.ldc) + col;
            if constexpr (MODE == M_FWD1_SWIGLU) {
              const float h1 = acc[i][q], h3 = acc3[i][q];
              if (p.H1) {
                reinterpret_cast<float*>(p.H1 + row * p.ldh)[col] = h1;
                reinterpret_cast<float*>(p.H3 + row * p.ldh)[col] = h3;
              }
              *c = h1 * sigm(h1) * h3;
            } else if constexpr (MODE == M_FWD1) {
              if (p.H1) reinterpret_cast<float*>(p.H1 + row * p.ldh)[col] = acc[i][q];
              *c = act_f(acc[i][q], p.act);
            } else if constexpr (MODE == M_BWD_DA_SWIGLU) {
              const float h1 = reinterpret_cast<const float*>(p.H1 + row * p.ldh)[col];
              const float h3 = reinterpret_cast<const float*>(p.H3 + row * p.ldh)[col];
              // d silu(h1) h3 / dh1 = h3 sg (1 + h1 (1 - sg)), d / dh3 = h1 sg
              const float sg = sigm(h1), x = acc[i][q] * sg, u = x * h3;
              *c = __builtin_fmaf(u, __builtin_fmaf(-h1, sg, h1), u);
              c[p.f] = x * h1;
            } else if constexpr (MODE == M_BWD_DA) {
              *c = acc[i][q] * act_grad_f(reinterpret_cast<const float*>(p.H1 + row * p.ldh)[col], p.act);
            } else {
              *c = acc[i][q];
            }
          }
        }
      }
    };
    if constexpr (VARK) {
      switch (t.h) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        default: run(std::integral_constant<int, 4>{}); break;
      }
    } else {
      switch (t.h) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 4: run(std::integral_constant<int, 4>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        default: run(std::integral_constant<int, 6>{}); break;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// transposed weights
// ---------------------------------------------------------------------------
// Transposed copy of expert weights (bf16), so that dX reads them
// K-contiguous: dst[g][n][k] = src1[g][k][n] for k < K1 and src2[g][k - K1][n]
// for K1 <= k < K1 + K2 (dst rows of K1 + K2 elements).  A workgroup moves a
// 64 (k) x 64 (n) block through LDS: 16-byte loads along n, 16-byte stores
// along k.  K1, K2 and N are multiples of 8, so no vector straddles an edge
// or the seam between the two sources.
constexpr int kTr = 64;
__global__ __launch_bounds__(256) void transpose_w_kernel(const uint16_t* __restrict__ src1,
                                                          const uint16_t* __restrict__ src2,
                                                          int K1, int K2, int N,
                                                          uint16_t* __restrict__ dst) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[kTr][kTr + 8];
  const int g = blockIdx.z;
  const int n0 = blockIdx.x * kTr;
  const int K = K1 + K2;
  const int64_t s1 = static_cast<int64_t>(g) * K1 * N, s2 = static_cast<int64_t>(g) * K2 * N;
  for (int k0 = blockIdx.y * kTr; k0 < K; k0 += gridDim.y * kTr) {
    __syncthreads();   // the previous block's reads of the tile are done
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = threadIdx.x + 256 * i;
      const int kk = c >> 3, nn = (c & 7) * 8;
      const int k = k0 + kk, n = n0 + nn;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (k < K && n < N) {
        const uint16_t* src = k < K1 ? src1 + s1 + static_cast<int64_t>(k) * N + n
                                     : src2 + s2 + static_cast<int64_t>(k - K1) * N + n;
        v = *reinterpret_cast<const uint4*>(src);
      }
      *reinterpret_cast<uint4*>(&tile[kk][nn]) = v;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = threadIdx.x + 256 * i;
      const int nn = c >> 3, kk = (c & 7) * 8;
      const int n = n0 + nn, k = k0 + kk;
      if (n < N && k < K) {
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          w[j] = static_cast<uint32_t>(tile[kk + 2 * j][nn]) |
                 (static_cast<uint32_t>(tile[kk + 2 * j + 1][nn]) << 16);
        *reinterpret_cast<uint4*>(dst + (static_cast<int64_t>(g) * N + n) * K + k) =
            make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// split-K reduction
// ---------------------------------------------------------------------------
// dW[g] = sum over the expert's split slots, in slot order, or zeros for an
// expert without rows.  A bounded grid strides over the elements (blockIdx.y =
// expert), so experts with one segment cost one early exit per block rather
// than a launch per 1024 elements.  The zeros are written here and not by the
// products' tiles: streamed, the 1 GB of 61 of 64 experts at 4096 x 1024 takes
// 154 us beside the sums, after the products of the others, where tiles of
// zeros among the products took about 190 us more (the product 325 -> 156 us,
// this kernel 29 -> 154 us).
constexpr int kReduceBlocks = 1024;   // blocks per expert

// The slots are added in slot order; their loads are issued four at a time
// ahead of the adds, so a thread waits out one memory latency per four slots.
__global__ __launch_bounds__(256) void split_reduce_kernel(
    const float* __restrict__ partial, int64_t slot_elems, const Sched* __restrict__ sc,
    float* __restrict__ dwA, float* __restrict__ dwB, int64_t dw_gstride, int split_row,
    int N) {
  const int g = blockIdx.y;
  const int ns = sc->nsplit[g];
  if (ns == 1) return;
  if (ns == 0) {
    const int64_t na = static_cast<int64_t>(split_row) * N;   // elements in dwA, the rest in dwB
    for (int64_t i = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 4; i < slot_elems;
         i += static_cast<int64_t>(gridDim.x) * 1024) {
      float* dst = i < na ? dwA + static_cast<int64_t>(g) * dw_gstride + i
                          : dwB + static_cast<int64_t>(g) * dw_gstride + (i - na);
      *reinterpret_cast<float4*>(dst) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    return;
  }
  const float* base = partial + static_cast<int64_t>(sc->slot0[g]) * slot_elems;
  auto add = [](float4& a, const float4& v) { a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w; };
  for (int64_t i = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 4; i < slot_elems;
       i += static_cast<int64_t>(gridDim.x) * 1024) {
    const float* p0 = base + i;
    float4 acc = *reinterpret_cast<const float4*>(p0);
    int sl = 1;
    for (; sl + 3 < ns; sl += 4) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        v[u] = *reinterpret_cast<const float4*>(p0 + static_cast<int64_t>(sl + u) * slot_elems);
#pragma unroll
      for (int u = 0; u < 4; ++u) add(acc, v[u]);
    }
    for (; sl < ns; ++sl) add(acc, *reinterpret_cast<const float4*>(p0 + static_cast<int64_t>(sl) * slot_elems));
    int64_t row, col;
    if (slot_elems < (int64_t(1) << 31)) {   // the usual case: 32-bit division
      const uint32_t ii = static_cast<uint32_t>(i);
      row = ii / static_cast<uint32_t>(N);
      col = ii % static_cast<uint32_t>(N);
    } else {
      row = i / N;
      col = i % N;
    }
    float* dst = row < split_row
                     ? dwA + static_cast<int64_t>(g) * dw_gstride + row * N + col
                     : dwB + static_cast<int64_t>(g) * dw_gstride + (row - split_row) * N + col;
    *reinterpret_cast<float4*>(dst) = acc;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
int persistent_grid() {
  const int n = num_cus();
  return (n + kXcds - 1) / kXcds * kXcds;
}

inline int cdiv(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

// [rows_alloc, f] planes of h_save: A (ReLU), H and A (GELU), H1, H3 and A
// (SwiGLU).
int h_save_planes(moe_act act) { return act == MOE_SWIGLU ? 3 : act == MOE_GELU_TANH ? 2 : 1; }

// Sizes of the schedule and of every workspace buffer.
struct FfnPlan {
  int E, d, f, F;            // F = f (relu/gelu) or 2f (swiglu)
  int64_t rows_alloc;
  int64_t rows_most;         // rows_alloc, or fewer (FfnFwd)
  size_t es;
  int max_mtiles, max_mid, max_segs, max_slots, tmn_min;
  int64_t slot_elems;
  // byte offsets inside the workspace
  size_t o_sched, o_mtile, o_mid, o_seg, o_end_sched;
  size_t o_abuf, o_dh, o_part, o_wt13, total_fwd, total_bwd, total_bwd_wt;
};

bool make_plan(moe_dtype dt, moe_act act, int E, int d, int f, int64_t rows_alloc, FfnPlan& pl) {
  if (!dtype_ok(dt) || E < 1 || E > kMaxE || !width_ok(d) || !width_ok(f) || !rows_ok(rows_alloc))
    return false;
  if (act != MOE_RELU && act != MOE_GELU_TANH && act != MOE_SWIGLU) return false;
  pl.E = E; pl.d = d; pl.f = f; pl.F = act == MOE_SWIGLU ? 2 * f : f;
  pl.rows_alloc = pl.rows_most = rows_alloc;
  pl.es = esize(dt);
  // every operand offset inside a 256-row tile (K-contiguous operands) or a
  // K step (K-major ones) stays below 2^31 bytes: buffer loads take 32-bit
  // offsets
  const int64_t max_ld = static_cast<int64_t>(pl.es) * (2 * static_cast<int64_t>(f) > d ? 2 * static_cast<int64_t>(f) : d);
  if (max_ld > kMaxOperandRowBytes) return false;
  pl.max_mtiles = cdiv(rows_alloc, BM) + E;
  pl.max_mid = cdiv(rows_alloc, kMidUnit) + E;
  const int tmn2 = cdiv(d, BM) * cdiv(f, BN);
  const int tmn13 = cdiv(pl.F, BM) * cdiv(d, BN);
  pl.tmn_min = tmn2 < tmn13 ? tmn2 : tmn13;
  const int64_t kcap = (rows_alloc + kKc - 1) / kKc * kKc + static_cast<int64_t>(kKc) * E;
  const int64_t slots_a = 1024 / pl.tmn_min;
  const int64_t slots_b = 2 * kcap / kSplitFloor;
  pl.max_slots = static_cast<int>(slots_a < slots_b ? slots_a : slots_b) + 1;
  pl.max_segs = E + pl.max_slots;
  pl.slot_elems = static_cast<int64_t>(pl.F) * d > static_cast<int64_t>(d) * f
                      ? static_cast<int64_t>(pl.F) * d : static_cast<int64_t>(d) * f;
  size_t o = 0;
  pl.o_sched = o; o = align_up(o + sizeof(Sched), 256);
  pl.o_mtile = o; o = align_up(o + sizeof(int2) * pl.max_mtiles, 256);
  pl.o_mid = o; o = align_up(o + 2 * sizeof(int2) * pl.max_mid, 256);
  pl.o_seg = o;   o = align_up(o + sizeof(int4) * pl.max_segs, 256);
  pl.o_end_sched = o;
  const size_t es = pl.es;
  // forward: the activation buffer A [rows_alloc, f] when no h_save is given
  pl.o_abuf = o;
  pl.total_fwd = align_up(o + static_cast<size_t>(rows_alloc) * f * es, 256);
  // backward: dH [rows_alloc, F] and the split partial sums
  o = pl.o_end_sched;
  pl.o_dh = o;   o = align_up(o + static_cast<size_t>(rows_alloc) * pl.F * es, 256);
  pl.o_part = o; o = align_up(o + static_cast<size_t>(pl.max_slots) * pl.slot_elems * 4, 256);
  pl.total_bwd = o;
  // bf16: room for the transposed copy of [W1; W3] that dX may read
  // ([E, d, F]: row n of expert e = [W1_e[:, n]; W3_e[:, n]])
  pl.o_wt13 = o;
  pl.total_bwd_wt = dt == MOE_BF16 ? align_up(o + static_cast<size_t>(E) * d * pl.F * es, 256) : o;
  return true;
}

// nt0, nt1: column tiles (of kMidN columns) of the call's products with N = f
// (K = d) and with N = d (K = k1), c0, c1: their K steps' times, for the
// heights of the two mid tile lists.
SchedArgs sched_args(const FfnPlan& pl, int nt0, int nt1, int k1, const StepCost& c0,
                     const StepCost& c1, char* ws) {
  const bool f32 = pl.es == 4;
  const int ks = f32 ? kF32Step : 64;
  return {pl.E, pl.rows_alloc, pl.max_mtiles, pl.max_mid, pl.max_segs, pl.tmn_min, pl.max_slots,
          {nt0, nt1}, {cdiv(pl.d, ks), cdiv(k1, ks)}, 2 * persistent_grid(),
          {f32 ? kStepF32 : c0, f32 ? kStepF32 : c1}, reinterpret_cast<Sched*>(ws + pl.o_sched),
          reinterpret_cast<int2*>(ws + pl.o_mtile), reinterpret_cast<int2*>(ws + pl.o_mid),
          reinterpret_cast<int4*>(ws + pl.o_seg)};
}

moe_status launch_schedule(hipStream_t s, const SchedArgs& a, const int32_t* offsets,
                           const int32_t* rows) {
  MOE_TIMED("ffn_schedule", s);
  schedule_kernel<<<1, 64 * kSchedTasks, 0, s>>>(offsets, rows, a);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

GemmParams base_params(const FfnPlan& pl, const int32_t* offsets, char* ws) {
  GemmParams p{};
  p.offsets = offsets;
  p.sched = reinterpret_cast<const Sched*>(ws + pl.o_sched);
  p.mtile = reinterpret_cast<const int2*>(ws + pl.o_mtile);
  p.seg = reinterpret_cast<const int4*>(ws + pl.o_seg);
  p.kmsplit = 0x7FFFFFFF;
  return p;
}

// Tile choice of the bf16 products (moe_set_gemm_tiles: 0 automatic, 1 the
// 256x256 kernel only, 2 the two-workgroups-per-CU kernel only).
int g_tile_mode = 0;

// mid_pays (tiles.hpp) for the forward and the data gradients; the weight
// gradients (K not known on the host) compare rounds, a round of 128x128 tiles
// taking 0.65 of one of 256x256 tiles.
bool use_mid_tiles(const FfnPlan& pl, moe_dtype dt, bool vark, bool gated, bool act, bool b_km,
                   const GemmParams& p) {
  if (dt == MOE_F32) return true;
  if (g_tile_mode == 1) return false;
  if (g_tile_mode == 2) return true;
  const int G = persistent_grid();
  if (vark) {
    const int64_t big = static_cast<int64_t>(pl.E) * cdiv(p.M_out, BM) * cdiv(p.N, BN);
    const int64_t mid = static_cast<int64_t>(pl.E) * cdiv(p.M_out, kMidDwH * kMidUnit) * cdiv(p.N, kMidN);
    return 13 * ((mid + 2 * G - 1) / (2 * G)) < 20 * ((big + G - 1) / G);
  }
  return mid_pays({pl.E, pl.rows_alloc, pl.rows_most, p.N, p.K, gated, act, b_km, p.lda, p.ldb}, G);
}

// dX with a transposed copy of [W1; W3] (moe_set_dx_weight_copy: 0
// automatic, 1 never, 2 always; bf16 only).  Read K-major, the weights need
// two transpose reads per MFMA fragment; read K-contiguous, dX ran 8-9%
// faster on 16384-row experts (same box, c5 and c4 shapes), and the copy
// moves 4 E d F bytes at about 5 TB/s.  The copy pays for itself from about
// 6000 rows per expert; the rule takes it from 8192 (rows_alloc / E: the
// row budget, as the host knows no fills).
int g_wt_mode = 0;
constexpr int64_t kWtRowsPerExpert = 8192;

bool use_wt13(const FfnPlan& pl, moe_dtype dt) {
  if (dt != MOE_BF16 || g_wt_mode == 1) return false;
  return g_wt_mode == 2 || pl.rows_alloc >= kWtRowsPerExpert * pl.E;
}

const char* pass_name(int pass) {
  static const char* names[] = {"gemm_fwd_h", "gemm_fwd_y", "gemm_bwd_da", "gemm_bwd_dx",
                                "gemm_bwd_dw2", "gemm_bwd_dw13", "gemm_bwd_dx"};
  return names[pass];
}

// Launches one product; sets the tile counts along N (and M for the weight
// gradients) for the kernel it picks.
template <int MODE, int PASS>
moe_status launch_gemm(hipStream_t s, moe_dtype dt, const FfnPlan& pl, char* ws, GemmParams p) {
  constexpr bool VARK = MODE == M_DW, GATED = MODE == M_FWD1_SWIGLU;
  constexpr bool ACTIVE = MODE != M_STORE && MODE != M_DW;
  const bool mid = use_mid_tiles(pl, dt, VARK, GATED, ACTIVE, b_layout(PASS) == L_KM, p);
  const int tn = mid ? kMidN : BN;
  p.ntiles = cdiv(p.N, GATED ? tn / 2 : tn);
  p.dw_h = kMidDwH;
  if constexpr (VARK) {
    // fp32 weight gradients: the highest tile that still gives every place of
    // the persistent grid one
    if (dt == MOE_F32)
      while (p.dw_h > 1 && static_cast<int64_t>(pl.E) * cdiv(p.M_out, p.dw_h * kMidUnit) * p.ntiles <
                               2 * persistent_grid())
        p.dw_h /= 2;
    p.mtiles_out = cdiv(p.M_out, mid ? p.dw_h * kMidUnit : BM);
  }
  // tile list 0: the products with N = f (H, dA); list 1: N = d (Y, dX)
  p.mid_list = PASS == P_FWD_H || PASS == P_BWD_DA ? 0 : 1;
  if (mid) p.mtile = reinterpret_cast<const int2*>(ws + pl.o_mid) + p.mid_list * static_cast<int64_t>(pl.max_mid);
  // the persistent grid, or fewer workgroups (a multiple of 8, for the XCD
  // mapping) when even the most tiles the schedule can list are fewer
  const int64_t max_items = VARK ? static_cast<int64_t>(pl.max_segs) * p.mtiles_out * p.ntiles
                                 : static_cast<int64_t>(mid ? pl.max_mid : pl.max_mtiles) *
                                       p.ntiles;
  const int64_t full = (mid ? 2 : 1) * static_cast<int64_t>(persistent_grid());
  const int grid = static_cast<int>(std::min(full, std::max<int64_t>(kXcds, (max_items + kXcds - 1) / kXcds * kXcds)));
  MOE_TIMED(pass_name(PASS), s);
  if (dt == MOE_F32) {
    if constexpr (PASS != P_BWD_DX_T) ffn_gemm_f32_kernel<MODE, PASS><<<grid, kThreads16, 0, s>>>(p);
  } else if (mid) {
    ffn_gemm16_mid_kernel<MODE, PASS><<<grid, kThreads16, 0, s>>>(p);
  } else {
    ffn_gemm16_kernel<MODE, PASS><<<grid, kThreads16, 0, s>>>(p);
  }
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

#define MOE_TRY(...)                       \
  do {                                     \
    moe_status st_ = (__VA_ARGS__);        \
    if (st_ != MOE_OK) return st_;         \
  } while (0)

// dW[g] = sum of expert g's split slots: rows [0, split_row) of the [M_out, N]
// result go to dwA, the rest to dwB; dw_gstride is the per-expert stride of
// dwA and dwB (f x d for [dW1; dW3], whose M_out is 2f under SwiGLU).
moe_status launch_split_reduce(hipStream_t s, const FfnPlan& pl, char* ws, int M_out, int N,
                               float* dwA, float* dwB, int split_row, int64_t dw_gstride) {
  const int64_t elems = static_cast<int64_t>(M_out) * N;
  const int64_t bx = cdiv(elems, 1024);
  dim3 grid(static_cast<unsigned>(bx < kReduceBlocks ? bx : kReduceBlocks), pl.E);
  MOE_TIMED("split_reduce", s);
  split_reduce_kernel<<<grid, 256, 0, s>>>(
      reinterpret_cast<const float*>(ws + pl.o_part), elems,
      reinterpret_cast<const Sched*>(ws + pl.o_sched), dwA, dwB, dw_gstride, split_row, N);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

// dst[g] = [src1[g]; src2[g]]^T for g < E (src1 [K1, N], src2 [K2, N] per expert).
moe_status launch_transpose_w(hipStream_t s, int E, const void* src1, const void* src2, int K1,
                              int K2, int N, void* dst) {
  const dim3 grid(cdiv(N, kTr), std::min(cdiv(K1 + K2, kTr), 32768), E);
  MOE_TIMED("transpose_w", s);
  transpose_w_kernel<<<grid, 256, 0, s>>>(static_cast<const uint16_t*>(src1),
                                          static_cast<const uint16_t*>(src2), K1, K2, N,
                                          static_cast<uint16_t*>(dst));
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

}  // namespace
}  // namespace moe

using namespace moe;

extern "C" moe_status moe_set_gemm_tiles(int mode) {
  if (mode < 0 || mode > 2) return MOE_EINVAL;
  g_tile_mode = mode;
  return MOE_OK;
}

extern "C" size_t moe_ffn_fwd_workspace_bytes(moe_dtype dt, moe_act act, int E, int d, int f,
                                              int64_t rows_alloc) {
  FfnPlan pl;
  return make_plan(dt, act, E, d, f, rows_alloc, pl) ? pl.total_fwd : 0;
}

extern "C" size_t moe_ffn_bwd_workspace_bytes(moe_dtype dt, moe_act act, int E, int d, int f,
                                              int64_t rows_alloc) {
  FfnPlan pl;
  if (!make_plan(dt, act, E, d, f, rows_alloc, pl)) return 0;
  return use_wt13(pl, dt) ? pl.total_bwd_wt : pl.total_bwd;
}

extern "C" moe_status moe_set_dx_weight_copy(int mode) {
  if (mode < 0 || mode > 2) return MOE_EINVAL;
  g_wt_mode = mode;
  return MOE_OK;
}

namespace moe {

moe_status ffn_fwd_check(const FfnFwd& a, size_t workspace_bytes) {
  FfnPlan pl;
  if (!make_plan(a.dt, a.act, a.E, a.d, a.f, a.rows_alloc, pl)) return MOE_EINVAL;
  if (!a.offsets || !a.rows || !a.w1 || !a.w2) return MOE_EINVAL;
  if (a.act == MOE_SWIGLU && !a.w3) return MOE_EINVAL;
  if (a.rows_alloc > 0 && (!a.x_disp || !a.y_disp)) return MOE_EINVAL;
  if (!aligned16(a.w1) || !aligned16(a.w2) || (a.w3 && !aligned16(a.w3)) ||
      (a.x_disp && !aligned16(a.x_disp)) || (a.y_disp && !aligned16(a.y_disp)) ||
      (a.h_save && !aligned16(a.h_save)))
    return MOE_EINVAL;
  if (a.rows_alloc == 0) return MOE_OK;
  if (!a.workspace || workspace_bytes < pl.total_fwd || !aligned16(a.workspace)) return MOE_EWORKSPACE;
  return MOE_OK;
}

SchedArgs ffn_fwd_sched(const FfnFwd& a) {
  FfnPlan pl;
  make_plan(a.dt, a.act, a.E, a.d, a.f, a.rows_alloc, pl);
  return sched_args(pl, cdiv(a.f, a.act == MOE_SWIGLU ? kMidN / 2 : kMidN), cdiv(a.d, kMidN), a.f,
                    step16(a.d * 2ll, a.d * 2ll, false), step16(a.f * 2ll, a.f * 2ll, false),
                    static_cast<char*>(a.workspace));
}

moe_status ffn_fwd_launch(hipStream_t s, const FfnFwd& a, bool scheduled) {
  if (a.rows_alloc == 0) return MOE_OK;
  FfnPlan pl;
  make_plan(a.dt, a.act, a.E, a.d, a.f, a.rows_alloc, pl);
  pl.rows_most = a.rows_most;
  if (!scheduled) MOE_TRY(launch_schedule(s, ffn_fwd_sched(a), a.offsets, a.rows));
  char* ws = static_cast<char*>(a.workspace);
  const moe_dtype dt = a.dt;
  const moe_act act = a.act;
  const int d = a.d, f = a.f;
  const int32_t* offsets = a.offsets;
  const int64_t rows_alloc = a.rows_alloc;
  const void *x_disp = a.x_disp, *w1 = a.w1, *w3 = a.w3, *w2 = a.w2;
  void *h_save = a.h_save, *y_disp = a.y_disp;
  const int64_t es = static_cast<int64_t>(pl.es);
  const int64_t plane = rows_alloc * f * es;   // one [rows_alloc, f] plane of h_save
  const bool sw = act == MOE_SWIGLU;
  // A = act(H): the last plane of h_save when the caller keeps activations.
  // ReLU keeps A alone (relu'(H) = [A > 0]), so H is never written there.
  const int h_planes = h_save_planes(act) - 1;
  char* abuf = h_save ? static_cast<char*>(h_save) + h_planes * plane : ws + pl.o_abuf;

  GemmParams p = base_params(pl, offsets, ws);
  p.A = static_cast<const char*>(x_disp);
  p.lda = d * es;
  p.B = static_cast<const char*>(w1);
  p.B2 = static_cast<const char*>(w3);
  p.ldb = d * es;
  p.b_gstride = static_cast<int64_t>(f) * d * es;
  p.K = d;
  p.N = f;
  p.act = act == MOE_RELU ? ACT_RELU : (act == MOE_GELU_TANH ? ACT_GELU : ACT_SWIGLU);
  p.C = abuf;
  p.ldc = f * es;
  p.H1 = h_planes > 0 ? static_cast<char*>(h_save) : nullptr;
  p.H3 = h_save && sw ? static_cast<char*>(h_save) + plane : nullptr;
  p.ldh = f * es;
  if (sw) MOE_TRY(launch_gemm<M_FWD1_SWIGLU, P_FWD_H>(s, dt, pl, ws, p));
  else MOE_TRY(launch_gemm<M_FWD1, P_FWD_H>(s, dt, pl, ws, p));

  GemmParams q = base_params(pl, offsets, ws);
  q.A = abuf;
  q.lda = f * es;
  q.B = static_cast<const char*>(w2);
  q.ldb = f * es;
  q.b_gstride = static_cast<int64_t>(d) * f * es;
  q.K = f;
  q.N = d;
  q.C = static_cast<char*>(y_disp);
  q.ldc = d * es;
  MOE_TRY(launch_gemm<M_STORE, P_FWD_Y>(s, dt, pl, ws, q));
  return MOE_OK;
}

}  // namespace moe

extern "C" moe_status moe_expert_ffn_fwd(void* stream, moe_dtype dt, moe_act act, int E, int d,
                                         int f, const int32_t* offsets, const int32_t* rows,
                                         int64_t rows_alloc, const void* x_disp, const void* w1,
                                         const void* w3, const void* w2, void* h_save,
                                         void* y_disp, void* workspace, size_t workspace_bytes) {
  const FfnFwd a = {dt, act, E, d, f, offsets, rows, rows_alloc, x_disp, w1, w3, w2, h_save,
                    y_disp, workspace, rows_alloc};
  MOE_TRY(ffn_fwd_check(a, workspace_bytes));
  return ffn_fwd_launch(static_cast<hipStream_t>(stream), a, false);
}

extern "C" moe_status moe_expert_ffn_bwd(void* stream, moe_dtype dt, moe_act act, int E, int d,
                                         int f, const int32_t* offsets, const int32_t* rows,
                                         int64_t rows_alloc, const void* x_disp,
                                         const void* h_save, const void* w1, const void* w3,
                                         const void* w2, const void* dy_disp, void* dx_disp,
                                         float* dw1, float* dw3, float* dw2, void* workspace,
                                         size_t workspace_bytes) {
  FfnPlan pl;
  if (!make_plan(dt, act, E, d, f, rows_alloc, pl)) return MOE_EINVAL;
  if (!offsets || !rows || !w1 || !w2 || !dw1 || !dw2) return MOE_EINVAL;
  if (act == MOE_SWIGLU && (!w3 || !dw3)) return MOE_EINVAL;
  if (rows_alloc > 0 && (!x_disp || !h_save || !dy_disp || !dx_disp)) return MOE_EINVAL;
  if (!aligned16(w1) || !aligned16(w2) || (w3 && !aligned16(w3)) || !aligned16(dw1) ||
      !aligned16(dw2) || (dw3 && !aligned16(dw3)) || (x_disp && !aligned16(x_disp)) ||
      (h_save && !aligned16(h_save)) || (dy_disp && !aligned16(dy_disp)) ||
      (dx_disp && !aligned16(dx_disp)))
    return MOE_EINVAL;
  if (!workspace || workspace_bytes < pl.total_bwd || !aligned16(workspace)) return MOE_EWORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  // dX reads [W1; W3] from a transposed copy (K-contiguous) when the rule
  // or the caller's setting asks for it and the workspace has room for it
  const bool wt = use_wt13(pl, dt) && workspace_bytes >= pl.total_bwd_wt;
  MOE_TRY(launch_schedule(s, sched_args(pl, cdiv(f, kMidN), cdiv(d, kMidN), pl.F,
                                        step16(d * 2ll, f * 2ll, true),
                                        step16(pl.F * 2ll, (wt ? pl.F : d) * 2ll, !wt), ws),
                          offsets, rows));
  const int64_t es = static_cast<int64_t>(pl.es);
  const bool sw = act == MOE_SWIGLU;
  const int F = pl.F;
  char* dh = ws + pl.o_dh;      // [rows_alloc, F]: dH, or [dH1 | dH3]
  const int actc = act == MOE_RELU ? ACT_RELU : (act == MOE_GELU_TANH ? ACT_GELU : ACT_SWIGLU);
  const int64_t plane = rows_alloc * f * es;
  // A = act(H), saved by the forward after H (or H1, H3); ReLU saves A alone
  // and its derivative reads A: relu'(H) = [H > 0] = [A > 0]
  const char* abuf = static_cast<const char*>(h_save) + (h_save_planes(act) - 1) * plane;
  const char* h1 = act == MOE_RELU ? abuf : static_cast<const char*>(h_save);
  const char* h3 = sw ? h1 + plane : nullptr;

  char* wt13 = ws + pl.o_wt13;
  if (wt) MOE_TRY(launch_transpose_w(s, E, w1, sw ? w3 : nullptr, f, sw ? f : 0, d, wt13));

  // dx_disp = [dH1 | dH3] [W1; W3]: from the transposed copy, or W1, W3 read
  // K-major (W3 from k = f on)
  auto launch_dx = [&]() -> moe_status {
    if (wt) {
      GemmParams q = base_params(pl, offsets, ws);
      q.A = dh;
      q.lda = F * es;
      q.B = wt13;
      q.ldb = F * es;
      q.b_gstride = static_cast<int64_t>(d) * F * es;
      q.K = F;
      q.N = d;
      q.C = static_cast<char*>(dx_disp);
      q.ldc = d * es;
      return launch_gemm<M_STORE, P_BWD_DX_T>(s, dt, pl, ws, q);
    }
    GemmParams q = base_params(pl, offsets, ws);
    q.A = dh;
    q.lda = F * es;
    q.B = static_cast<const char*>(w1);
    q.B2 = sw ? static_cast<const char*>(w3) : nullptr;
    q.kmsplit = sw ? f : 0x7FFFFFFF;
    q.ldb = d * es;
    q.b_gstride = static_cast<int64_t>(f) * d * es;
    q.K = F;
    q.N = d;
    q.C = static_cast<char*>(dx_disp);
    q.ldc = d * es;
    return launch_gemm<M_STORE, P_BWD_DX>(s, dt, pl, ws, q);
  };
  // Order of the four products: dA first (it writes dH), dX right after it,
  // except when dx_disp is small enough to stay in the last-level cache: then
  // dX goes last, so the dispatch backward that follows reads dx_disp from
  // that cache rather than from HBM.
  const bool dx_last = rows_alloc * d * es <= kDxLastBytes;

  // dA = dY W2 (W2 read K-major: its rows are the d inputs) -> dH
  GemmParams p = base_params(pl, offsets, ws);
  p.A = static_cast<const char*>(dy_disp);
  p.lda = d * es;
  p.B = static_cast<const char*>(w2);
  p.ldb = f * es;
  p.b_gstride = static_cast<int64_t>(d) * f * es;
  p.K = d;
  p.N = f;
  p.act = actc;
  p.C = dh;
  p.ldc = F * es;
  p.H1 = const_cast<char*>(h1);
  p.H3 = const_cast<char*>(h3);
  p.ldh = f * es;
  p.f = f;
  if (sw) MOE_TRY(launch_gemm<M_BWD_DA_SWIGLU, P_BWD_DA>(s, dt, pl, ws, p));
  else MOE_TRY(launch_gemm<M_BWD_DA, P_BWD_DA>(s, dt, pl, ws, p));
  if (!dx_last) MOE_TRY(launch_dx());

  // dW2 [d, f] = dY^T A, contracting over each expert's dispatched rows
  GemmParams r = base_params(pl, offsets, ws);
  r.A = static_cast<const char*>(dy_disp);
  r.lda = d * es;
  r.M_out = d;
  r.B = abuf;
  r.ldb = f * es;
  r.N = f;
  r.dwA = dw2;
  r.dwB = dw2;
  r.dw_gstride = static_cast<int64_t>(d) * f;
  r.split_row = d;
  r.partial = reinterpret_cast<float*>(ws + pl.o_part);
  r.slot_elems = static_cast<int64_t>(d) * f;
  MOE_TRY(launch_gemm<M_DW, P_BWD_DW2>(s, dt, pl, ws, r));
  MOE_TRY(launch_split_reduce(s, pl, ws, d, f, dw2, dw2, d, r.dw_gstride));

  // [dW1; dW3] [F, d] = [dH1 dH3]^T X
  GemmParams u = base_params(pl, offsets, ws);
  u.A = dh;
  u.lda = F * es;
  u.M_out = F;
  u.B = static_cast<const char*>(x_disp);
  u.ldb = d * es;
  u.N = d;
  u.dwA = dw1;
  u.dwB = sw ? dw3 : dw1;
  u.dw_gstride = static_cast<int64_t>(f) * d;
  u.split_row = f;
  u.partial = reinterpret_cast<float*>(ws + pl.o_part);
  u.slot_elems = static_cast<int64_t>(F) * d;
  MOE_TRY(launch_gemm<M_DW, P_BWD_DW13>(s, dt, pl, ws, u));
  MOE_TRY(launch_split_reduce(s, pl, ws, F, d, dw1, sw ? dw3 : dw1, f, u.dw_gstride));

  // dx_disp last when it fits the last-level cache (see kDxLastBytes)
  if (dx_last) MOE_TRY(launch_dx());
  return MOE_OK;
}
