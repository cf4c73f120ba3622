// LM-head forward (logits + vocab-chunked online log-sum-exp + sampled-token gather),
// the GRPO/DAPO/GSPO loss coefficient, and the LM-head backward, for gfx950.
//
// Sec. 3.2 (post-pruning evaluation) and Sec. 3.1 (Eq. 1, Eq. grad).  With P the softmax
// of z = H W^T and g = dL/dlogp:  dZ = g (onehot(y) - P),  dH = dZ W,  dW = dZ^T H.
//
// One tiled GEMM kernel does the three contractions.  C[m, n] = sum_k A[m, k] B[n, k]
// with operands moved by direct global->LDS loads:
//   bf16: 256 x 256 block tiles, 8 wavefronts of 128 x 64, v_mfma_f32_16x16x32_bf16, 64-wide K
//         steps, the two wavefronts of a SIMD multiplying in turn;
//   f32:  v_mfma_f32_32x32x2_f32, 32-wide K steps; logits tiles of 256 vocab rows x 64 tokens,
//         gradient tiles of 64 x 64 or 128 x 128 (f32_gemm_kernel).
// Work is cut into slabs of whole sequences; per slab:
//   FWD  C = W . H_slab^T  (rows = vocab, cols = tokens, K = d).  Epilogue: per token,
//        the block's max and sum exp(z - s_t) over its 256 vocab rows (in-lane over 32
//        values, two lane-row swaps, one LDS exchange), the sampled token's logit, and
//        E1[t][v] = exp(z - s_t) (s_t = 0 unless exp(z) would leave float range).
//   merge   partials -> lse, logp, row max; rows whose max is too far from s_t get
//           s_t = max_t and their token block is evaluated again (rare; the loss kernel merges them).
//   loss    g_t and c_t = g_t exp(s_t - lse_t) per token (one block per sequence).  With a
//           backward it also folds the one-hot term into the exp-logits: since
//           g_t = c_t exp(lse_t - s_t), E1[t][y_t] -= exp(lse_t - s_t) makes
//           c_t E1[t][v] = g_t (P[t][v] - [v = y_t]) = -dZ[t][v] for every v.
//   DH   C = E1 . W^T  (rows = tokens, cols = d, K = vocab):  dH[t] = -c_t C[t].
//   DW   with B = c_t H[t] (K = tokens): bf16 computes C' = Bd . E1 (Bd = B^T; rows = d, cols =
//        vocab; E1 is read K-major through transposing LDS reads), f32 computes C = E1^T . B
//        (rows = vocab, cols = d; both read K-major):  dW[v] (+)= -C[v].
// Nothing of size [T, V] exists: the exp-logit buffer holds one slab, [slab, V], and the
// default slab (32768 tokens) does not grow with T.
#include <algorithm>
#include <cstdlib>
#include <mutex>
#include <string>
#include <vector>

#include "common.h"

namespace fastrl {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kBM = 256, kBN = 256;
constexpr int kThreads = 512;  // of a bf16 GEMM block: 8 wavefronts, two per SIMD

// MODE_DWT: the bf16 dW GEMM computed transposed, dW^T = Bd E (rows = hidden columns, cols =
// vocab rows, K = tokens), so that it runs on the 8-wavefront engine with E as a K-major B
// MODE_DHT: the bf16 dhidden GEMM of small calls, which reads W itself (K-major, K = vocab) instead
// of a transposed copy and can cut its long K into parts (launch_bwd_direct)
enum GemmMode { MODE_FWD = 0, MODE_DH = 1, MODE_DW = 2, MODE_DWT = 3, MODE_DHT = 4 };

struct GemmParams {
  const void* A;            // [M, lda]
  int64_t lda;
  int32_t M;
  const void* B;            // [N rows, ldb] (rows via b_rows when non-null)
  int64_t ldb;
  int32_t N;
  const int32_t* b_rows;    // FWD: row_index (nullable) offset to the slab
  int64_t b_row_base;       // FWD: first kept token of the slab
  int32_t K;
  int32_t nmb, nnb;         // block grid (M blocks, N blocks)
  int32_t group;            // tile order: M-blocks per sweep over the N-blocks (tile_group)
  int32_t tail, pieces;     // FWD: the last `tail` whole tiles are cut into `pieces` (fwd_tiles)
  int32_t narrow;           // FWD: 64-token columns of the narrow last tile column (0: none)
  int32_t block0;           // float32: tile number of a launch's first block
  // ---- FWD epilogue
  float* pmax;              // [nmb][ldp]
  float* psum;              // [nmb][ldp]
  float* psz;               // [nmb][ldp] or NULL: sum of exp(z - ref) * z (entropy)
  int64_t ldp;
  float* zlab;              // [slab]
  const int32_t* yslab;     // [slab] label of each slab token (-1: invalid)
  const float* shift;       // [slab] s_t (nullable = 0)
  void* E1;                 // [slab rows][ldE1 = V_pad]   E1[t][v] = exp(z[t][v] - s_t)
  int64_t ldE1;
  int32_t Vreal;
  int32_t store_e;          // 0: partials only, 1: partials + E, 2: same for redo blocks
  const int32_t* redo_blk;  // [nnb] token blocks to evaluate again (store_e == 2)
  const int32_t* redo_any;  // nonzero iff some token block of the slab is marked
  // ---- DH epilogue
  int32_t ksplit;           // DHT: parts of K (1: none)
  int32_t part_first;       // DHT: blocks take the parts of a tile in a row (dh_ksplit)
  float* part;              // DHT with ksplit > 1: [ksplit][M][d] float32 sums of each part
  void* dH;                 // [.., d] at slab offset
  int32_t dH_bf16;
  const float* cslab;       // [slab]
  int32_t d;
  // ---- DW epilogue
  float* dW;                // [V, d]
  int32_t dW_acc;           // add to dW (later slabs) instead of overwriting it
};

// Tile order: consecutive blocks are dealt round-robin to the 8 XCDs and run at about the same
// time, so the order of logical tiles decides which operand strips are in use together.  A group
// of M-blocks shares each sweep over the N-blocks (p.group, chosen per shape on the host by
// tile_group).  Logits GEMM (short K): 32 at d = 3584, so each XCD holds 4 vocab blocks x 8
// token blocks of the 256 tiles in flight and all XCDs read the same 8 hidden row blocks.
// Backward GEMMs (long K): 4 at d = 3584; all XCDs walk neighbouring tiles through K together,
// so a strip that several XCDs read is fetched once into the shared last-level cache (giving
// each XCD its own contiguous range of tiles measured 2-4% slower here).
template <int MODE>
__device__ __forceinline__ void tile_coords(int& mb, int& nb, int nmb, int nnb, int b, int group) {
  // the groups are vocab blocks in both dW forms: M blocks of MODE_DW, N blocks of MODE_DWT
  constexpr bool GN = MODE == MODE_DWT;
  const int ng = GN ? nnb : nmb, ns = GN ? nmb : nnb;
  const int per_group = group * ns;
  const int gid = b / per_group;
  const int first = gid * group;
  const int gsz = min(ng - first, group);
  const int in = b % per_group;
  const int a = first + in % gsz, sweep = in / gsz;
  mb = GN ? sweep : a;
  nb = GN ? a : sweep;
}

typedef __attribute__((address_space(3))) void lds_void_t;

// bf16 main loop of the logits GEMM (z = W h: A = LM-head rows, B = gathered hidden rows, K = d),
// the dhidden GEMM (A = the slab's exp-logit rows, B = W^T rows or, K-major, W itself, K = padded
// vocab) and the transposed dW GEMM (A = Bd rows, B = the exp-logit tile read K-major, K = padded
// slab).  A tile of 256 x 64 NJ (NJ < 4: logits only), K in tiles of 64; eight wavefronts, each a
// 128 x 16 NJ part on v_mfma_f32_16x16x32_bf16 (8 x NJ accumulators of 16 x 16; lane l holds rows
// 4 (l / 16) .. + 3 of column l % 16).
//
// The two wavefronts of a SIMD (wm = 0, 1) take turns: in one phase one of them multiplies a whole
// K tile out of registers (64 MFMAs), with the loads of later tiles issued in between, while the
// other reads the 24 fragments of its next K tile from LDS; a barrier, and they swap.  So a matrix
// core is always fed by one wavefront that waits for nothing, and LDS reads and the rendezvous are
// hidden behind the other one's MFMAs.  (When both ran MFMAs and reads interleaved in step, with one
// rendezvous per K tile, the matrix cores were busy 68% of the time at 1.85 GHz; so, 79% at 1.73 GHz
// under the same power limit.  Logits of 27136 tokens at 7B 21.9 -> 20.5 ms, loss call of 27000
// tokens 68.3 -> 63.8 ms, 507 tokens at d = 1536 1061 -> 914 us.  With the loads in the reading
// phase, that phase outlasted the other's MFMAs: 61% busy, 22.4 ms.)  The barrier that ends a
// multiplying phase comes before its last MFMAs, which cover its latency.
//
// LDS: two stages of A (32 KB each) and three of B.  Wavefronts wm = 0 read tile k in phase 2k and
// multiply it in phase 2k + 1, wm = 1 one phase later.  Loads (global_load_lds_dwordx4, 1 KB an
// instruction, lane l into 16-byte slot l) go out in a multiplying phase, as soon as their stage is
// free: in the phase of tile k, wm = 0 loads the A rows it reads itself (0 .. 127) of tile k + 2 and
// half of B of tile k + 2; wm = 1 its A rows (128 .. 255) of tile k + 2 and the other half of B of
// tile k + 3.  The end of the next multiplying phase waits for them: two phases later.
//
// LDS layout (rows of 64 k = 128 B): row r keeps its k-chunk c (8 bf16) in slot
// c ^ ((r >> 1) & 7).  The LDS serves a 16-byte-per-lane read 16 lanes (256 B, 64 banks) at a
// time, and rows r..r+15 of a fragment then land on 16 distinct 16-byte bank groups; the
// swizzle is applied on the global side (each lane loads the chunk that belongs in its slot).
// A K-major B tile is 64 k-rows of 256 columns (512 B), column chunk c of row k in slot c ^ swz(k),
// swz(k) = ((k & 3) << 1) | (((k >> 3) & 1) << 3).
constexpr int kStage = kBM * 64;                          // elements of one operand's stage
constexpr int kSmemBytes = (2 + 3) * kStage * 2;          // 160 KB: all of a compute unit's LDS
// LDS that no wavefront reads or loads into any more once one of them is past its last K tile:
// the A stage of the tile before the last (of nk)
__device__ __forceinline__ uint16_t* free_stage(uint16_t* smem, int nk) {
  return smem + (nk & 1) * kStage;
}
// Off, Step: a lane's offset and a K tile's, in bytes; of 64 bits for rows of kMaxLd elements or more
// (lm_wide_kernel).
template <int MODE, int NJ = 4, typename Off = uint32_t, typename Step = int>
__device__ __forceinline__ void mainloop_bf16(const GemmParams& p, int m0, int n0,
                                              f32x4_t (&acc)[8][NJ], uint16_t* smem, int kt0 = 0,
                                              int nkt = 0) {
  static_assert(NJ == 4 || MODE == MODE_FWD, "narrow tiles: logits only");
  constexpr int BK = 64;
  constexpr bool DHT = MODE == MODE_DHT;
  constexpr bool BKM = MODE == MODE_DWT || DHT;  // B stored K-major (B[n][k] at k * ldb + n)
  constexpr bool GATHER = MODE == MODE_FWD;      // B rows through b_rows
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const char* Ag = static_cast<const char*>(p.A);
  const char* Bg = static_cast<const char*>(p.B);
  uint16_t* const sA = smem;
  uint16_t* const sB = smem + 2 * kStage;
  const int K = p.K;
  const int nk = DHT ? nkt : (K + BK - 1) / BK;
  // ---- loads.  Addresses are a uniform base (the first of a load's rows) plus a lane offset (32 bits)
  // in bytes; gathered rows take 64-bit lane addresses.  Rows past the edge load a valid one (their
  // results are never stored).
  const int lrow = lane >> 3;
  const int gch = (lane & 7) ^ (lrow >> 1);  // k-chunk of an even load; of an odd one gch ^ 4
  const char* abase[4];
  Off aoff[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r0 = min(m0 + wave * 32 + j * 8, p.M - 1);
    abase[j] = Ag + 2 * int64_t(r0) * p.lda;
    aoff[j] = 2u * Off(min(r0 + lrow, p.M - 1) - r0) * Off(p.lda);
    if constexpr (MODE != MODE_FWD) aoff[j] += 16u * uint32_t(gch ^ ((j & 1) << 2));
  }
  const char* bbase[NJ];  // uniform (not gathered) or lane address
  Off boff[NJ];
  const int bodd = (NJ & 1) ? (wave & 1) : 0;  // load j of B: an odd one if j + bodd is
  uint32_t bhi = 0;
  if constexpr (BKM) {
    // load j fills k-rows 8 wave + 2 j and the next: lane l slot l % 32 of the first or second
    bhi = (lane >> 5) ? 2u * uint32_t(p.ldb) : 0u;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int k = wave * 8 + 2 * j + (lane >> 5);
      const int n = (((lane & 31) ^ (((k & 3) << 1) | (((k >> 3) & 1) << 3))) << 3);
      // (W's rows end at N: columns past it load a valid chunk)
      boff[j] = 2u * uint32_t(DHT ? min(n, p.N - 8 - n0) : n);
      if constexpr (!DHT) boff[j] += bhi;
      bbase[j] = Bg + 2 * int64_t(n0);
    }
  } else if constexpr (GATHER) {
    int64_t bi[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      bi[j] = min(n0 + (wave * NJ + j) * 8 + lrow, p.N - 1) + p.b_row_base;
    if (p.b_rows) {  // the index loads are issued together: one memory round trip
      int32_t g[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) g[j] = __builtin_nontemporal_load(p.b_rows + bi[j]);
#pragma unroll
      for (int j = 0; j < NJ; ++j) bi[j] = g[j];
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) bbase[j] = Bg + 2 * bi[j] * p.ldb;
  } else {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int r0 = min(n0 + (wave * NJ + j) * 8, p.N - 1);
      bbase[j] = Bg + 2 * int64_t(r0) * p.ldb;
      boff[j] = 2u * Off(min(r0 + lrow, p.N - 1) - r0) * Off(p.ldb) +
                16u * uint32_t(gch ^ ((j & 1) << 2));
    }
  }
  // byte offset of a lane's chunk inside tile kt (logits: K need not be whole tiles, and a partial
  // last tile loads a valid chunk for those past K)
  auto chunk = [&](int kt, int odd) { return 2 * min((gch ^ (odd << 2)) * 8, K - 8 - kt * BK); };
  auto issue_a = [&](int kt, int st) {
    uint16_t* d = sA + st * kStage + wave * 32 * BK;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      Off o = aoff[j];
      if constexpr (MODE == MODE_FWD) o += uint32_t(chunk(kt, j & 1));
      const char* base = abase[j] + int64_t(DHT ? kt + kt0 : kt) * (2 * BK);
      const char* src = base + o;
      __builtin_amdgcn_global_load_lds(src, (lds_void_t*)(d + j * 8 * BK), 16, 0, 0);
    }
  };
  auto issue_b = [&](int kt, int st) {
    uint16_t* d = sB + st * kStage + wave * NJ * 8 * BK;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const char* src;
      if constexpr (BKM) {
        int k = (DHT ? kt + kt0 : kt) * BK + wave * 8 + 2 * j;
        Off o = boff[j];
        if constexpr (DHT) {  // vocab rows past the end load the last one (their exp-logits are 0)
          if (k + 1 < p.Vreal) o += bhi;
          k = min(k, p.Vreal - 1);
        }
        src = bbase[j] + 2 * int64_t(k) * p.ldb + o;
      } else if constexpr (GATHER) {
        src = bbase[j] + (Step(kt) * (2 * BK) + chunk(kt, (j + bodd) & 1));
      } else {
        src = bbase[j] + int64_t(kt) * (2 * BK) + boff[j];
      }
      __builtin_amdgcn_global_load_lds(src, (lds_void_t*)(d + j * 8 * BK), 16, 0, 0);
    }
  };
  // ---- fragments of a whole K tile: A rows wm*128 + i*16 + (lane & 15), B rows wn*16 NJ + j*16 +
  // (lane & 15), k-chunk 4 kk + lane / 16 (8 consecutive k per lane) of the 32-k step kk
  bf16x8_t fa[2][8], fb[2][NJ];
  const int sw = ((lane & 15) >> 1) & 7;  // ((row >> 1) & 7) of the fragment rows this lane reads
  const int slot0 = ((lane >> 4) ^ sw) * 8, slot1 = ((4 + (lane >> 4)) ^ sw) * 8;
  const int afo = (wm * 128 + (lane & 15)) * BK, bfo = (wn * 16 * NJ + (lane & 15)) * BK;
  // K-major B fragments (ds_read_b64_tr_b16): in 16-lane group g, lane jj reads 4 n of k-row
  // 8 g + 4 s + jj / 4 (s = first / second 4 k of the lane's 8) at n = 16 j + 4 (jj % 4) of
  // the wavefront's 64 columns, and receives the 4 k of column n = 16 j + jj.  The row swizzle
  // puts the 8 rows that lanes 0-31 (and 32-63) read on 16 distinct 16-byte bank groups.  They are
  // inline assembly: before the builtin form the compiler waits for every outstanding direct-to-LDS
  // load.  frag_wait waits for them, and passes them on as operands so that no use precedes it.
  uint32_t bfa[4];  // LDS byte addresses of this lane's K-major B fragments in stage 0
  if constexpr (BKM) {
    typedef __attribute__((address_space(3))) const uint16_t lds_u16_t;
    const int g = lane >> 4, jj = lane & 15;
    const int swz = ((jj >> 2) << 1) | ((g & 1) << 3);  // swz of the rows this lane reads
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = wn * 64 + 16 * j + 4 * (jj & 3);
      const int o = (8 * g + (jj >> 2)) * kBN + (((n >> 3) ^ swz) << 3) + (n & 7);
      bfa[j] = uint32_t(uintptr_t((lds_u16_t*)(sB + o)));
    }
  }
  auto read_frags = [&](int sta, int stb) {
    const uint16_t* as = sA + sta * kStage + afo;
    const uint16_t* bs = sB + stb * kStage + bfo;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int slot = kk ? slot1 : slot0;
      if constexpr (BKM) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
          u32x2_t h0, h1;
          const uint32_t a = bfa[j] + uint32_t(stb) * (kStage * 2);
          if (kk == 0) {
            asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(h0) : "v"(a) : "memory");
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:2048" : "=v"(h1) : "v"(a) : "memory");
          } else {
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:16384" : "=v"(h0) : "v"(a) : "memory");
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:18432" : "=v"(h1) : "v"(a) : "memory");
          }
          fb[kk][j] = __builtin_bit_cast(bf16x8_t, u32x4_t{h0[0], h0[1], h1[0], h1[1]});
        }
      } else {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          fb[kk][j] = *reinterpret_cast<const bf16x8_t*>(bs + j * 16 * BK + slot);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i)
        fa[kk][i] = *reinterpret_cast<const bf16x8_t*>(as + i * 16 * BK + slot);
    }
  };
  auto frag_wait = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (BKM)
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(fb[0][0]), "+v"(fb[0][1]), "+v"(fb[0][2]), "+v"(fb[0][3]),
                     "+v"(fb[1][0]), "+v"(fb[1][1]), "+v"(fb[1][2]), "+v"(fb[1][3])
                   :
                   : "memory");
    else
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };
  auto barrier = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mma = [&](int kk, int i0, int i1) {
#pragma unroll
    for (int i = i0; i < i1; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[kk][i], fb[kk][j], acc[i][j], 0, 0, 0);
  };
  // ---- prologue: what the multiplying phases of tiles -2 and -1 (and -3) would have loaded
  if (wm == 0) {
    issue_a(0, 0);
    issue_b(0, 0);
    if (nk > 1) {
      issue_a(1, 1);
      issue_b(1, 1);
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 + NJ) : "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    barrier();
  } else {
    issue_b(0, 0);
    issue_a(0, 0);
    if (nk > 2) {
      issue_b(1, 1);
      issue_a(1, 1);
      issue_b(2, 2);
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 + 2 * NJ) : "memory");  // B of tile 0
      barrier();
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 + NJ) : "memory");
      barrier();
    } else {
      if (nk > 1) {
        issue_b(1, 1);
        issue_a(1, 1);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      barrier();
      barrier();
    }
  }
  int sb = 0, sbl = wm ? 0 : 2;  // B stages of tile k and of the tile whose B is loaded
  // full: tile k + 3 exists; last: k == nk - 1
  auto tile = [&](int k, auto full_c, auto last_c) {
    constexpr bool FULL = decltype(full_c)::value, LAST = decltype(last_c)::value;
    // reading phase
    read_frags(k & 1, sb);
    frag_wait();
    barrier();
    if constexpr (LAST && MODE == MODE_FWD) {
      // a partial last tile: nothing past K
      if ((K % BK) != 0) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const bool past = k * BK + (4 * kk + (lane >> 4)) * 8 >= K;
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (past) fa[kk][i] = bf16x8_t{};
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            if (past) fb[kk][j] = bf16x8_t{};
        }
      }
    }
    // multiplying phase; before its barrier the loads of the multiplying phase before have landed
    __builtin_amdgcn_s_setprio(1);
    if constexpr (!LAST) {
      if (FULL || k + 2 < nk) issue_a(k + 2, k & 1);
      if (FULL || k + 2 + wm < nk) issue_b(k + 2 + wm, sbl);
    }
    mma(0, 0, 8);
    mma(1, 0, 7);
    if constexpr (FULL) {
#pragma unroll
      for (int q = 0; q < 4 + NJ; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, NJ, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 15 * NJ - (4 + NJ) * NJ, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!LAST) {
      if (FULL || k + 2 + wm < nk) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 + NJ) : "memory");
      else if (k + 2 < nk) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    if (!LAST || wm == 0) barrier();
    mma(1, 7, 8);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    sb = sb == 2 ? 0 : sb + 1;
    sbl = sbl == 2 ? 0 : sbl + 1;
  };
  int k = 0;
  for (; k + 3 < nk; ++k) tile(k, std::true_type{}, std::false_type{});
  for (; k + 1 < nk; ++k) tile(k, std::false_type{}, std::false_type{});
  tile(k, std::false_type{}, std::true_type{});
}

// Reductions over the four 16-lane groups of a wavefront (lanes c, c + 16, c + 32, c + 48) with
// row swaps instead of LDS-routed shuffles: a 16-lane-row swap of x with itself leaves rows
// (r0, r0, r2, r2) and (r1, r1, r3, r3), whose sum is the xor-16 partner sum; a half swap then
// does the same for xor 32.  Each step adds the same two operands as the xor shuffle would.
__device__ __forceinline__ float group_sum4(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

__device__ __forceinline__ float group_max4(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Epilogue of the bf16 logits GEMM (16 x 16 accumulator tiles: acc[i][j] covers vocab rows
// wm*128 + 16 i .. +15 and tokens wn*16 NJ + 16 j .. +15; lane l holds rows 4 (l / 16) + q of
// token column l % 16).  Per token column: the block's max over its vocab rows, the sampled
// token's logit, and with a stored exp (store_e != 0) E[t][v] = exp(z - s_t) with the sums
// sum exp(z - s_t) and sum exp(z - s_t) z; without one (old / ref log-probs), the sums relative
// to the block max.  A column's 256 rows are spread over the 4 lane groups of two wavefronts:
// lane-row swaps, then one LDS exchange between the wavefronts.
template <int NJ>
__device__ __forceinline__ void fwd_epilogue_bf16(const GemmParams& p, int m0, int n0, int mb,
                                                  f32x4_t (&acc)[8][NJ], uint16_t* smem) {
  // (the cross-wave exchange takes LDS that the main loop has done with)
  float* xmax = reinterpret_cast<float*>(free_stage(smem, (p.K + 63) / 64));  // [2 wm][256 cols]
  float* xsum = xmax + 2 * kBN;
  float* xsz = xsum + 2 * kBN;
  constexpr int NT = kThreads;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int g = lane >> 4, c = lane & 15;
  const int Vr = p.Vreal;
  const bool rel = p.store_e != 0;
  const bool rows_full = m0 + kBM <= Vr;  // every vocab row of this block exists
  const int rbase = m0 + wm * 128 + 4 * g;  // vocab row of acc[i][j][q]: rbase + 16 i + q
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int cl = wn * 16 * NJ + j * 16 + c;
    const int t = n0 + cl;  // slab token
    const bool tok_ok = t < p.N;
    const int y = tok_ok ? p.yslab[t] : -1;
    // columns past the slab store exp(z - inf) = 0
    const float s_t = tok_ok ? (p.shift ? p.shift[t] : 0.0f) : INFINITY;
    // max over the lane's 32 rows in four independent chains; a full vocab block (all but the
    // last) takes a branch without the row test, so the chains become three-input maxima
    float mxp[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (rows_full) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) mxp[i & 3] = fmaxf(mxp[i & 3], acc[i][j][q]);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          mxp[i & 3] = fmaxf(mxp[i & 3], rbase + 16 * i + q < Vr ? acc[i][j][q] : -INFINITY);
    }
    float mx = fmaxf(fmaxf(mxp[0], mxp[1]), fmaxf(mxp[2], mxp[3]));
    // the sampled token's logit: held by one lane group of one wavefront (rare per column)
    const int dy = y - m0 - wm * 128;
    if (dy >= 0 && dy < 128 && ((dy >> 2) & 3) == g) {
      float zl = 0.0f;
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) zl = (16 * i + q == (dy & ~12)) ? acc[i][j][q] : zl;
      p.zlab[t] = zl;
    }
    mx = group_max4(mx);
    if (g == 0) xmax[wm * kBN + cl] = mx;
    if (rel) {
      uint16_t* e1 = static_cast<uint16_t*>(p.E1) + int64_t(t) * p.ldE1;
      // exp(z - s_t) = exp2(z log2e - s_t log2e): one FMA and v_exp_f32 per logit (s_t = +inf
      // past the slab gives 0).  Two uniform choices get code of their own, since this pass is
      // most of the epilogue (a per-block timing probe: 8.5% of the kernel): the row check only
      // in the last vocab block, the z-weighted sum only when the entropy is asked for.
      const float sl = s_t * 1.4426950408889634f;
      auto pass = [&](auto full_c, auto z_c) {
        constexpr bool FULL = decltype(full_c)::value, WZ = decltype(z_c)::value;
        float ssp[4] = {0.0f, 0.0f, 0.0f, 0.0f}, zsp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ip = 0; ip < 4; ++ip) {  // tile pair 2 ip, 2 ip + 1
          uint32_t pk[2][2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int i = 2 * ip + h;
            float e[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              e[q] = __builtin_amdgcn_exp2f(fmaf(acc[i][j][q], 1.4426950408889634f, -sl));
              if (!FULL && rbase + 16 * i + q >= Vr) e[q] = 0.0f;
              ssp[ip] += e[q];
              if (WZ) zsp[ip] = fmaf(e[q], acc[i][j][q], zsp[ip]);
            }
            typedef float f32x2_t __attribute__((ext_vector_type(2)));
            typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
            pk[h][0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{e[0], e[1]}, bf16x2_t));
            pk[h][1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{e[2], e[3]}, bf16x2_t));
          }
          // lane group g holds rows 4 g .. 4 g + 3 of both tiles; one swap between the groups
          // of each 32-lane half (odd group's tile-2ip rows <-> even group's tile-2ip+1 rows)
          // leaves group g with 8 consecutive rows: tile 2 ip + (g & 1), rows 8 (g >> 1) .. + 7
#pragma unroll
          for (int w = 0; w < 2; ++w) {
            const auto sw = __builtin_amdgcn_permlane16_swap(pk[0][w], pk[1][w], false, false);
            pk[0][w] = sw[0];
            pk[1][w] = sw[1];
          }
          const int v0 = m0 + wm * 128 + (2 * ip + (g & 1)) * 16 + (g >> 1) * 8;
          *reinterpret_cast<uint4*>(e1 + v0) = make_uint4(pk[0][0], pk[0][1], pk[1][0], pk[1][1]);
        }
        float ssum = (ssp[0] + ssp[1]) + (ssp[2] + ssp[3]);
        ssum = group_sum4(ssum);
        if (g == 0) xsum[wm * kBN + cl] = ssum;
        if constexpr (WZ) {
          float zsum = (zsp[0] + zsp[1]) + (zsp[2] + zsp[3]);
          zsum = group_sum4(zsum);
          if (g == 0) xsz[wm * kBN + cl] = zsum;
        }
      };
      if (rows_full) {
        if (p.psz) pass(std::true_type{}, std::true_type{});
        else pass(std::true_type{}, std::false_type{});
      } else {
        if (p.psz) pass(std::false_type{}, std::true_type{});
        else pass(std::false_type{}, std::false_type{});
      }
    }
  }
  __syncthreads();
  if (!rel) {
    // sums relative to the block's column max M: exp(z - M) = exp2(z log2e - M log2e), one FMA
    // and one v_exp_f32 per logit; as in the stored-exp pass, full vocab blocks skip the row
    // test and the z-weighted sum is only formed when the entropy is asked for
    auto pass = [&](auto full_c, auto z_c) {
      constexpr bool FULL = decltype(full_c)::value, WZ = decltype(z_c)::value;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int cl = wn * 16 * NJ + j * 16 + c;
        const float ml = fmaxf(xmax[cl], xmax[kBN + cl]) * 1.4426950408889634f;
        float ssp[4] = {0.0f, 0.0f, 0.0f, 0.0f}, zsp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float ex = __builtin_amdgcn_exp2f(fmaf(acc[i][j][q], 1.4426950408889634f, -ml));
            if (!FULL && rbase + 16 * i + q >= Vr) ex = 0.0f;
            ssp[i & 3] += ex;
            if (WZ) zsp[i & 3] = fmaf(ex, acc[i][j][q], zsp[i & 3]);
          }
        float ssum = (ssp[0] + ssp[1]) + (ssp[2] + ssp[3]);
        ssum = group_sum4(ssum);
        if (g == 0) xsum[wm * kBN + cl] = ssum;
        if constexpr (WZ) {
          float zsum = (zsp[0] + zsp[1]) + (zsp[2] + zsp[3]);
          zsum = group_sum4(zsum);
          if (g == 0) xsz[wm * kBN + cl] = zsum;
        }
      }
    };
    if (rows_full) {
      if (p.psz) pass(std::true_type{}, std::true_type{});
      else pass(std::true_type{}, std::false_type{});
    } else {
      if (p.psz) pass(std::false_type{}, std::true_type{});
      else pass(std::false_type{}, std::false_type{});
    }
    __syncthreads();
  }
  for (int cl = tid; cl < 64 * NJ; cl += NT) {
    const int t = n0 + cl;
    if (t < p.N) {
      p.pmax[int64_t(mb) * p.ldp + t] = fmaxf(xmax[cl], xmax[kBN + cl]);
      p.psum[int64_t(mb) * p.ldp + t] = xsum[cl] + xsum[kBN + cl];
      if (p.psz) p.psz[int64_t(mb) * p.ldp + t] = xsz[cl] + xsz[kBN + cl];
    }
  }
}


// Epilogue of the bf16 dhidden GEMM on the 16 x 16 layout (acc[i][j]: token rows wm*128 + 16 i
// + 4 (l / 16) + q, hidden columns wn*64 + 16 j + l % 16): dH[t] = -c_t C[t] (the one-hot term
// is already in E1).
__device__ __forceinline__ void dh_epilogue_bf16(const GemmParams& p, int m0, int n0,
                                                 f32x4_t (&acc)[8][4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int g = lane >> 4, c = lane & 15;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = m0 + wm * 128 + 16 * i + 4 * g + q;
      if (t < p.M) {
        const float ct = p.cslab[t];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int n = n0 + wn * 64 + 16 * j + c;
          if (n < p.N) {
            const float val = -ct * acc[i][j][q];
            const int64_t o = int64_t(t) * p.d + n;
            if (p.dH_bf16) static_cast<uint16_t*>(p.dH)[o] = f32_to_bf16(val);
            else static_cast<float*>(p.dH)[o] = val;
          }
        }
      }
    }
}

// One part of a dhidden tile whose K is cut: the plain float32 sums.
__device__ __forceinline__ void dh_part_epilogue_bf16(const GemmParams& p, int m0, int n0, int s,
                                                      f32x4_t (&acc)[8][4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int g = lane >> 4, c = lane & 15;
  float* out = p.part + int64_t(s) * p.M * p.d;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = m0 + wm * 128 + 16 * i + 4 * g + q;
      if (t < p.M) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int n = n0 + wn * 64 + 16 * j + c;
          if (n < p.N) out[int64_t(t) * p.d + n] = acc[i][j][q];
        }
      }
    }
}

// Epilogue of the bf16 dW GEMM computed transposed (C' = Bd E on the 16 x 16 layout: acc[i][j]
// holds hidden columns n = wm*128 + 16 i + 4 (l / 16) + q of vocab row v = wn*64 + 16 j + l % 16):
// each lane owns 4 consecutive n of one dW row and moves them as one 16-byte access.
// dW[v][n] (+)= -C'[n][v] (the one-hot term is already in E1).  Needs d % 4 == 0 and a 16-byte
// aligned dW (checked on the host).
__device__ __forceinline__ void dwt_epilogue_bf16(const GemmParams& p, int m0, int n0,
                                                  f32x4_t (&acc)[8][4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int nq = m0 + wm * 128 + 4 * (lane >> 4);  // first hidden column of acc[0][j]
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int v = n0 + wn * 64 + 16 * j + (lane & 15);
    if (v < p.N) {
      f32x4_t* row = reinterpret_cast<f32x4_t*>(p.dW + int64_t(v) * p.d);
      // every load of the row first, so that their latencies overlap
      f32x4_t prev[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int n = nq + 16 * i;
        prev[i] = (p.dW_acc && n < p.M) ? row[n >> 2] : f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int n = nq + 16 * i;
        if (n < p.M) row[n >> 2] = prev[i] - acc[i][j];
      }
    }
  }
}

// one logits tile of 256 vocab rows x 64 NJ tokens
template <int NJ, typename Off = uint32_t, typename Step = int>
__device__ __forceinline__ void fwd_tile(const GemmParams& p, int mb, int n0, uint16_t* smem) {
  f32x4_t acc[8][NJ];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  mainloop_bf16<MODE_FWD, NJ, Off, Step>(p, mb * kBM, n0, acc, smem);
  fwd_epilogue_bf16<NJ>(p, mb * kBM, n0, mb, acc, smem);
}

// The tiles of a logits GEMM (fwd_tiles), in tile order over p.nnb columns: the last `tail` are cut
// into 64- or 128-token pieces; with p.narrow the last column is 64 p.narrow tokens wide.  Up to
// kMixCols columns the narrow tiles run among the others of their vocab block, which share its rows
// of W (read again from HBM otherwise); beyond, they run last and fill the final wave.  token_logprob
// with 80 tokens in the narrow column, us, last / among the others: d = 1536 336 tokens 220 / 185, 2128
// 831 / 810, 3152 1194 / 1172, 4176 1539 / 1536, 12368 4381 / 4407, 20560 7270 / 7336; d = 3584 336
// 452 / 395, 2128 1770 / 1740, 2640 2173 / 2160, 3152 (13 columns) 2557 / 2564, 5200 4068 / 4157, 20560
// 15630 / 16120.
constexpr int kMixCols = 12;
__device__ __forceinline__ void fwd_block(const GemmParams& p, int b, uint16_t* smem) {
  const bool own = p.narrow && p.nnb > kMixCols;  // narrow column after all others
  const int cols = p.nnb - (own ? 1 : 0);
  const int whole = p.nmb * cols - p.tail;
  int mb, nb, piece = -1;
  if (own && b >= whole) {
    mb = b - whole;
    nb = cols;
  } else {
    if (b >= whole) {
      piece = (b - whole) % p.pieces;
      b = whole + (b - whole) / p.pieces;
    }
    tile_coords<MODE_FWD>(mb, nb, p.nmb, cols, b, p.group);
  }
  const int n0 = nb * kBN;
  if (piece >= 0) {
    if (p.pieces == 2) fwd_tile<2>(p, mb, n0 + 128 * piece, smem);
    else fwd_tile<1>(p, mb, n0 + 64 * piece, smem);
  } else if (p.narrow && nb == p.nnb - 1) {
    if (p.narrow == 1) fwd_tile<1>(p, mb, n0, smem);
    else if (p.narrow == 2) fwd_tile<2>(p, mb, n0, smem);
    else fwd_tile<3>(p, mb, n0, smem);
  } else {
    fwd_tile<4>(p, mb, n0, smem);
  }
}

// the bf16 GEMMs (T is uint16_t)
template <typename T, int MODE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void lm_gemm_kernel(const GemmParams p) {
  static_assert(sizeof(T) == 2, "float32 runs f32_gemm_kernel");
  __shared__ __attribute__((aligned(1024))) char smem_raw[kSmemBytes];
  uint16_t* smem = reinterpret_cast<uint16_t*>(smem_raw);
  if constexpr (MODE == MODE_FWD) {
    fwd_block(p, blockIdx.x, smem);
  } else {
    int mb, nb;
    tile_coords<MODE>(mb, nb, p.nmb, p.nnb, blockIdx.x, p.group);
    const int m0 = mb * kBM, n0 = nb * kBN;
    f32x4_t acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    mainloop_bf16<MODE>(p, m0, n0, acc, smem);
    if constexpr (MODE == MODE_DH) dh_epilogue_bf16(p, m0, n0, acc);
    else dwt_epilogue_bf16(p, m0, n0, acc);
  }
}

// ------------------------------------------------------------------ float32 GEMMs
// C[m, n] = sum_k A[m, k] B[n, k] on v_mfma_f32_32x32x2_f32 (64 cycles each, so a wavefront needs
// little operand traffic and the tiles can be small): wavefronts as WM x WN over a BM x BN tile,
// 32-wide K steps, ST LDS stages filled by direct global->LDS loads ST - 1 steps ahead.  Float32
// problems are small (parity runs), so the grid has to fill the chip and the chain of K steps per
// block has to be short: 256 x 256 tiles with register-staged loads gave 3 blocks of 256 steps
// (1090 us) on the 640-token dhidden of d = 256, V = 4096, where these take 22 us.  Loss call with
// both gradients, 256 x 256 tiles -> these: 300 tokens (d 256, V 4096) 1376 -> 86 us, 2048 (512,
// 8192) 3000 -> 524, 2048 (1024, 32000) 11.0 -> 3.6 ms, 4096 (3584, 152064) 118.7 -> 118.2 ms; and
// with two logits wavefronts per SIMD and no test between a K tile's steps 76 us, 483 us, 3.36 ms,
// and 64.7 -> 58.8 ms for 2048 (3584, 152064).
//   FWD (A = W, B = gathered hidden rows): both K-contiguous, 256 x 64, so that the partials have
//        the same 256-row blocks as bf16; 8 wavefronts, two per SIMD, of 64 x 32.  In groups of 8
//        vocab blocks per sweep over the tokens (tile_coords), whose rows of W the columns share: one
//        column after the other, each read all of W again (token_logprob of 2500 tokens at d = 1536,
//        V = 151936 10.93 ms, 9.58 so; 2048 at 7B 20.3 -> 17.9; groups of 4 to 64 level).
//   DH  (A = E1, B[n][k] = W[k][n]): B K-major; K in p.ksplit parts (dh_reduce_kernel adds them).
//   DW  (A[v][t] = E1[t][v], B[n][t] = c_t H[t][n]): both K-major.
// Fragments: in step s of a tile, lane l of half h = l / 32 holds k = 8 s + 4 h + j for the j-th of
// four MFMAs.  K-contiguous rows are 128 bytes, 16-byte chunk c kept in slot c ^ ((row >> 1) & 7):
// one 16-byte read gives the four k, conflict-free over 16 rows.  K-major rows hold BM (or BN)
// columns, chunk c in slot c ^ (((k >> 2) & 1) << 3): the two halves of a 4-byte read (k and k + 4)
// fall on different banks.
template <int MODE, int BM, int BN, int WM, int WN, int ST>
__global__ __launch_bounds__(64 * WM * WN) void f32_gemm_kernel(const GemmParams p) {
  constexpr bool AKM = MODE == MODE_DW, BKM = MODE != MODE_FWD;
  constexpr int BK = 32, MI = BM / WM / 32, NI = BN / WN / 32;
  constexpr int ASZ = BM * BK, STAGE = (BM + BN) * BK;   // floats
  constexpr int NW = WM * WN;
  constexpr int LA = BM / (8 * NW), LB = BN / (8 * NW);  // loads per wavefront and tile
  static_assert(LB > 0 && (MODE != MODE_FWD || WM == 4) && STAGE * ST * 4 <= 160 * 1024, "");
  __shared__ __attribute__((aligned(16))) float smem[STAGE * ST];
  if (MODE == MODE_FWD && p.store_e == 2 && p.redo_any[0] == 0) return;
  const int nt = p.nmb * p.nnb;
  const int tile = p.block0 + int(blockIdx.x);
  const int part = MODE == MODE_DH ? tile / nt : 0;
  const int b = tile - part * nt;
  int mb = b % p.nmb, nb = b / p.nmb;
  if constexpr (MODE == MODE_FWD) tile_coords<MODE_FWD>(mb, nb, p.nmb, p.nnb, b, p.group);
  const int m0 = mb * BM, n0 = nb * BN;
  if (MODE == MODE_FWD && p.store_e == 2 && p.redo_blk[n0 / kBN] == 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const float* Ag = static_cast<const float*>(p.A);
  const float* Bg = static_cast<const float*>(p.B);
  const int nk_all = (p.K + BK - 1) / BK;
  const int kt0 = MODE == MODE_DH ? int(int64_t(nk_all) * part / p.ksplit) : 0;
  const int nk = MODE == MODE_DH ? int(int64_t(nk_all) * (part + 1) / p.ksplit) - kt0 : nk_all;
  // K-contiguous operand: load j of this wavefront fills rows 8 (wave L + j) + lane / 8; K-major:
  // 256 / cols k-rows.  Rows and columns past the matrix load valid ones (results not stored).
  int64_t abase[LA], bbase[LB];
#pragma unroll
  for (int j = 0; j < LA; ++j) {
    if constexpr (AKM) abase[j] = 0;
    else abase[j] = int64_t(min(m0 + 8 * (wave * LA + j) + (lane >> 3), p.M - 1)) * p.lda;
  }
#pragma unroll
  for (int j = 0; j < LB; ++j) {
    if constexpr (BKM) {
      bbase[j] = 0;
    } else {
      int64_t r = min(n0 + 8 * (wave * LB + j) + (lane >> 3), p.N - 1) + p.b_row_base;
      if (p.b_rows) r = p.b_rows[r];
      bbase[j] = r * p.ldb;
    }
  }
  auto issue = [&](int kt, int stage) {
    float* sa = smem + stage * STAGE + wave * LA * 256;
    float* sb = smem + stage * STAGE + ASZ + wave * LB * 256;
    const int kb = (kt0 + kt) * BK;
    auto kcontig = [&](const float* g, int64_t base, int row, float* dst) {
      // (chunks past a partial last tile load a valid one and are not read)
      const int k = min(kb + (((lane & 7) ^ ((row >> 1) & 7)) << 2), p.K - 4);
      __builtin_amdgcn_global_load_lds(g + base + k, (lds_void_t*)dst, 16, 0, 0);
    };
    auto kmajor = [&](const float* g, int64_t ld, int kmax, int c0, int cmax, int cols, int j, float* dst) {
      const int cpr = cols / 4, rpl = 64 / cpr;  // chunks per row, rows per load
      const int k = j * rpl + lane / cpr;
      const int c = ((lane % cpr) ^ (((k >> 2) & 1) << 3)) << 2;
      __builtin_amdgcn_global_load_lds(g + int64_t(min(kb + k, kmax)) * ld + min(c0 + c, cmax),
                                       (lds_void_t*)dst, 16, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < LA; ++j) {
      if constexpr (AKM) kmajor(Ag, p.lda, p.K - 1, m0, int(p.lda) - 4, BM, wave * LA + j, sa + j * 256);
      else kcontig(Ag, abase[j], 8 * (wave * LA + j) + (lane >> 3), sa + j * 256);
    }
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      if constexpr (BKM)
        kmajor(Bg, p.ldb, MODE == MODE_DH ? p.Vreal - 1 : p.K - 1, n0, p.N - 4, BN, wave * LB + j,
               sb + j * 256);
      else kcontig(Bg, bbase[j], 8 * (wave * LB + j) + (lane >> 3), sb + j * 256);
    }
  };
  const int l31 = lane & 31, half = lane >> 5;
  f32x16_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = f32x16_t{};
  // the four k of step s for row / column r of the tile
  auto frag = [&](bool km, const float* t, int r, int cols, int s) {
    if (km) {
      const int k = 8 * s + 4 * half;
      const float* q = t + k * cols + (r ^ (half << 5));
      return f32x4_t{q[0], q[cols], q[2 * cols], q[3 * cols]};
    }
    return *reinterpret_cast<const f32x4_t*>(t + r * BK + (((2 * s + half) ^ ((r >> 1) & 7)) << 2));
  };
  constexpr int PF = ST - 1;  // tiles in flight
#pragma unroll
  for (int i = 0; i < PF; ++i)
    if (i < nk) issue(i, i);
  for (int kt = 0; kt < nk; ++kt) {
    // own loads of tile kt have landed (later tiles' may be in flight), then everybody's have and
    // nobody reads the stage that the next load fills
    // (a plain s_barrier: __syncthreads would also wait for the later tiles' loads)
    if (kt + PF <= nk) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((PF - 1) * (LA + LB)) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt + PF < nk) issue(kt + PF, (kt + PF) % ST);
    const float* as = smem + (kt % ST) * STAGE;
    const float* bs = as + ASZ;
    auto step = [&](int s) {
      f32x4_t fa[MI], fb[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) fa[i] = frag(AKM, as, wm * (BM / WM) + i * 32 + l31, BM, s);
#pragma unroll
      for (int j = 0; j < NI; ++j) fb[j] = frag(BKM, bs, wn * (BN / WN) + j * 32 + l31, BN, s);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][q], fb[j][q], acc[i][j], 0, 0, 0);
    };
    const int ns = (p.K - (kt0 + kt) * BK + 7) / 8;  // below 4 in a partial last tile of the logits
    if (MODE != MODE_FWD || ns >= 4) {
      // (no test between the steps: the reads of a step go out among the MFMAs of the one before)
#pragma unroll
      for (int s = 0; s < 4; ++s) step(s);
    } else {
#pragma clang loop unroll(disable)
      for (int s = 0; s < ns; ++s) step(s);
    }
  }
  // acc[i][j][r]: row 32 i + 8 (r / 4) + 4 half + r % 4, column 32 j + l31 of the wavefront's part
  const int rw = wm * (BM / WM) + 4 * half, cw = wn * (BN / WN) + l31;
  if constexpr (MODE == MODE_FWD) {
    // per token column: the block's max and sum of exp, E1 and the sampled token's logit, as in
    // fwd_epilogue_bf16; a column's 256 rows are spread over the two halves of four wavefronts
    __syncthreads();  // LDS operand buffers are reused for the cross-wave exchange
    float* xmax = smem;  // [4][BN]
    float* xsum = xmax + WM * BN;
    float* xsz = xsum + WM * BN;
    const int Vr = p.Vreal;
    const bool rel = p.store_e != 0;
    auto row = [&](int i, int r) { return m0 + rw + 32 * i + 8 * (r >> 2) + (r & 3); };
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int cl = cw + 32 * j, t = n0 + cl;
      const bool tok_ok = t < p.N;
      const int y = tok_ok ? p.yslab[t] : -1;
      // columns past the slab store exp(z - inf) = 0
      const float s_t = tok_ok ? (p.shift ? p.shift[t] : 0.0f) : INFINITY;
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          mx = fmaxf(mx, row(i, r) < Vr ? acc[i][j][r] : -INFINITY);
          if (row(i, r) == y) p.zlab[t] = acc[i][j][r];
        }
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      if (half == 0) xmax[wm * BN + cl] = mx;
      if (rel) {
        float ssp[4] = {0.0f, 0.0f, 0.0f, 0.0f}, zsp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        float* e1 = static_cast<float*>(p.E1) + int64_t(t) * p.ldE1;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int rg = 0; rg < 4; ++rg) {
            float e[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float z = acc[i][j][rg * 4 + q];
              e[q] = row(i, rg * 4 + q) < Vr ? __expf(z - s_t) : 0.0f;
              ssp[rg] += e[q];
              zsp[rg] = fmaf(e[q], z, zsp[rg]);
            }
            *reinterpret_cast<float4*>(e1 + row(i, rg * 4)) = make_float4(e[0], e[1], e[2], e[3]);
          }
        float ssum = (ssp[0] + ssp[1]) + (ssp[2] + ssp[3]);
        float zsum = (zsp[0] + zsp[1]) + (zsp[2] + zsp[3]);
        ssum += __shfl_xor(ssum, 32, 64);
        zsum += __shfl_xor(zsum, 32, 64);
        if (half == 0) {
          xsum[wm * BN + cl] = ssum;
          xsz[wm * BN + cl] = zsum;
        }
      }
    }
    __syncthreads();
    auto col_max = [&](int cl) {
      return fmaxf(fmaxf(xmax[cl], xmax[BN + cl]), fmaxf(xmax[2 * BN + cl], xmax[3 * BN + cl]));
    };
    if (!rel) {
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int cl = cw + 32 * j;
        const float M = col_max(cl);
        float ssp[4] = {0.0f, 0.0f, 0.0f, 0.0f}, zsp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float z = acc[i][j][r];
            if (row(i, r) < Vr) {
              const float ex = __expf(z - M);
              ssp[r >> 2] += ex;
              zsp[r >> 2] = fmaf(ex, z, zsp[r >> 2]);
            }
          }
        float ssum = (ssp[0] + ssp[1]) + (ssp[2] + ssp[3]);
        float zsum = (zsp[0] + zsp[1]) + (zsp[2] + zsp[3]);
        ssum += __shfl_xor(ssum, 32, 64);
        zsum += __shfl_xor(zsum, 32, 64);
        if (half == 0) {
          xsum[wm * BN + cl] = ssum;
          xsz[wm * BN + cl] = zsum;
        }
      }
      __syncthreads();
    }
    if (tid < BN && n0 + tid < p.N) {
      const int64_t o = int64_t(mb) * p.ldp + n0 + tid;
      auto sum4 = [&](const float* x) {
        return (x[tid] + x[BN + tid]) + (x[2 * BN + tid] + x[3 * BN + tid]);
      };
      p.pmax[o] = col_max(tid);
      p.psum[o] = sum4(xsum);
      if (p.psz) p.psz[o] = sum4(xsz);
    }
  } else {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      auto row = [&](int r) { return m0 + rw + 32 * i + 8 * (r >> 2) + (r & 3); };
      // the loads of 16 rows first, so that their latencies overlap
      float prev[16][NI];
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const int n = n0 + cw + 32 * j;
          if constexpr (MODE == MODE_DH)
            prev[r][j] = p.ksplit == 1 && row(r) < p.M ? -p.cslab[row(r)] : 1.0f;
          else
            prev[r][j] = p.dW_acc && row(r) < p.M && n < p.N ? p.dW[int64_t(row(r)) * p.d + n] : 0.0f;
        }
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const int n = n0 + cw + 32 * j;
          if (row(r) >= p.M || n >= p.N) continue;
          const int64_t o = int64_t(row(r)) * p.d + n;
          if constexpr (MODE == MODE_DH) {
            const float v = prev[r][j] * acc[i][j][r];
            if (p.ksplit > 1) p.part[int64_t(part) * p.M * p.d + o] = v;
            else if (p.dH_bf16) static_cast<uint16_t*>(p.dH)[o] = f32_to_bf16(v);
            else static_cast<float*>(p.dH)[o] = v;
          } else {  // dW[v] (+)= -C[v] (the one-hot term is already in E1)
            p.dW[o] = prev[r][j] - acc[i][j][r];
          }
        }
    }
  }
}

// The two bf16 backward GEMMs of one slab in one launch: blocks [0, q.nmb q.nnb) are dhidden
// tiles (K = padded vocabulary), the rest transposed-dW tiles (K = padded slab, about five times
// shorter at the 7B shape).  Dispatched in block order, the dW tiles take the compute units that
// the last partial wave of dhidden tiles leaves idle (a 27K-token slab has 5.8 waves of
// dhidden tiles, a 19K-token slab at d = 1536 only 1.7).
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void lm_bwd_kernel(const GemmParams q, const GemmParams r) {
  __shared__ __attribute__((aligned(1024))) char smem_raw[kSmemBytes];
  uint16_t* smem = reinterpret_cast<uint16_t*>(smem_raw);
  const int nh = q.nmb * q.nnb;
  const int b = blockIdx.x;
  int mb, nb;
  f32x4_t acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  if (b < nh) {
    tile_coords<MODE_DH>(mb, nb, q.nmb, q.nnb, b, q.group);
    mainloop_bf16<MODE_DH>(q, mb * kBM, nb * kBN, acc, smem);
    dh_epilogue_bf16(q, mb * kBM, nb * kBN, acc);
  } else {
    tile_coords<MODE_DWT>(mb, nb, r.nmb, r.nnb, b - nh, r.group);
    mainloop_bf16<MODE_DWT>(r, mb * kBM, nb * kBN, acc, smem);
    dwt_epilogue_bf16(r, mb * kBM, nb * kBN, acc);
  }
}

// The same two GEMMs for calls of few tokens (direct_dh): dhidden reads W itself, K-major, with
// K cut into q.ksplit parts.  With few tokens there are few dhidden tiles but each has the whole
// vocabulary as K: one block per tile is a chain of V / 64 steps of ~1.2 us on a handful of
// compute units (12 of 256 at 507 tokens, d = 1536).  A part's float32 sums go to q.part and
// dh_reduce_kernel adds them in part order.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void lm_bwd_direct_kernel(const GemmParams q, const GemmParams r) {
  __shared__ __attribute__((aligned(1024))) char smem_raw[kSmemBytes];
  uint16_t* smem = reinterpret_cast<uint16_t*>(smem_raw);
  const int nt = q.nmb * q.nnb, nh = nt * q.ksplit;
  const int b = blockIdx.x;
  int mb, nb;
  f32x4_t acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  if (b < nh) {
    const int s = q.part_first ? b % q.ksplit : b / nt;
    tile_coords<MODE_DH>(mb, nb, q.nmb, q.nnb, q.part_first ? b / q.ksplit : b % nt, q.group);
    const int nk = q.K / 64;
    const int k0 = int(int64_t(nk) * s / q.ksplit), k1 = int(int64_t(nk) * (s + 1) / q.ksplit);
    mainloop_bf16<MODE_DHT>(q, mb * kBM, nb * kBN, acc, smem, k0, k1 - k0);
    if (q.ksplit > 1) dh_part_epilogue_bf16(q, mb * kBM, nb * kBN, s, acc);
    else dh_epilogue_bf16(q, mb * kBM, nb * kBN, acc);
  } else {
    tile_coords<MODE_DWT>(mb, nb, r.nmb, r.nnb, b - nh, r.group);
    mainloop_bf16<MODE_DWT>(r, mb * kBM, nb * kBN, acc, smem);
    dwt_epilogue_bf16(r, mb * kBM, nb * kBN, acc);
  }
}

// dH[t] = -c_t sum_s part[s][t], parts added in order; 4 columns per thread (d is a multiple of 8)
__global__ __launch_bounds__(256) void dh_reduce_kernel(const float* __restrict__ part,
                                                        int32_t ksplit, int32_t Tc, int32_t d,
                                                        const float* __restrict__ cslab,
                                                        void* __restrict__ dH, int32_t dH_bf16) {
  const int64_t n4 = int64_t(Tc) * (d / 4);
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n4) return;
  const f32x4_t* p4 = reinterpret_cast<const f32x4_t*>(part) + i;
  f32x4_t a = p4[0];
#pragma unroll 4
  for (int s = 1; s < ksplit; ++s) a += p4[int64_t(s) * n4];
  const float c = -cslab[i / (d / 4)];
  if (reinterpret_cast<uintptr_t>(dH) & 15u) {  // a caller's dhidden aligned to its elements only
    for (int e = 0; e < 4; ++e) {
      if (dH_bf16) static_cast<uint16_t*>(dH)[4 * i + e] = f32_to_bf16(c * a[e]);
      else static_cast<float*>(dH)[4 * i + e] = c * a[e];
    }
  } else if (dH_bf16) {
    const uint32_t lo = uint32_t(f32_to_bf16(c * a[0])) | uint32_t(f32_to_bf16(c * a[1])) << 16;
    const uint32_t hi = uint32_t(f32_to_bf16(c * a[2])) | uint32_t(f32_to_bf16(c * a[3])) << 16;
    static_cast<uint2*>(dH)[i] = make_uint2(lo, hi);
  } else {
    static_cast<f32x4_t*>(dH)[i] = f32x4_t{c * a[0], c * a[1], c * a[2], c * a[3]};
  }
}

// Second evaluation of the bf16 logits tiles whose token block holds a row that needs a shift:
// at most one block per compute unit walks the tiles in grid order and evaluates those of marked
// token blocks (store_e == 2); with no row marked, the usual case, every block returns at once.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void lm_redo_kernel(const GemmParams p) {
  if (p.redo_any[0] == 0) return;
  __shared__ __attribute__((aligned(1024))) char smem_raw[kSmemBytes];
  uint16_t* smem = reinterpret_cast<uint16_t*>(smem_raw);
  const int nt = p.nmb * p.nnb;
  for (int b = blockIdx.x; b < nt; b += gridDim.x) {
    int mb, nb;
    tile_coords<MODE_FWD>(mb, nb, p.nmb, p.nnb, b, p.group);
    if (p.redo_blk[nb] == 0) continue;  // the same for the whole block
    fwd_tile<4>(p, mb, nb * kBN, smem);
    __syncthreads();  // the epilogue's LDS exchange is read before the next tile's loads land
  }
}

// The bf16 GEMMs over rows of kMaxLd elements or more, one 256 x 256 tile a block: logits (also their
// second evaluation), dhidden from W^T or from W itself (K whole), transposed dW.
template <int MODE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void lm_wide_kernel(const GemmParams p) {
  __shared__ __attribute__((aligned(1024))) char smem_raw[kSmemBytes];
  uint16_t* smem = reinterpret_cast<uint16_t*>(smem_raw);
  int mb, nb;
  tile_coords<MODE>(mb, nb, p.nmb, p.nnb, blockIdx.x, p.group);
  if constexpr (MODE == MODE_FWD) {
    if (p.store_e == 2 && (p.redo_any[0] == 0 || p.redo_blk[nb] == 0)) return;
    fwd_tile<4, uint64_t, int64_t>(p, mb, nb * kBN, smem);
  } else {
    const int m0 = mb * kBM, n0 = nb * kBN;
    f32x4_t acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    mainloop_bf16<MODE, 4, uint64_t, int64_t>(p, m0, n0, acc, smem, 0, p.K / 64);
    if constexpr (MODE == MODE_DWT) dwt_epilogue_bf16(p, m0, n0, acc);
    else dh_epilogue_bf16(p, m0, n0, acc);
  }
}

// ------------------------------------------------------------------ small kernels

// s_t = 0, labels of the slab, validity; also clears the slab's flags (at most Tc + 1 of them) and,
// on a call's first slab, its count of rows evaluated again
__global__ __launch_bounds__(256) void slab_prep_kernel(
    const int32_t* __restrict__ token_ids, const int32_t* __restrict__ row_index, int64_t row_base,
    int32_t Tc, int32_t V, int32_t* __restrict__ yslab, float* __restrict__ shift,
    int32_t* __restrict__ status, int32_t* __restrict__ flags, int32_t nflags,
    int32_t* __restrict__ count) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < nflags) flags[t] = 0;
  if (t == 0 && count) count[0] = 0;
  if (t >= Tc) return;
  int64_t row = row_base + t;
  if (row_index) row = row_index[row];
  int y = token_ids[row];
  if (y < 0 || y >= V) {
    set_status(status, FASTRL_SB_BAD_TOKEN);
    y = -1;
  }
  yslab[t] = y;
  if (shift) shift[t] = 0.0f;
}

// partials -> lse, logp.  A block handles 32 tokens in SLICES slices of the vocabulary blocks (slice s
// takes blocks s, s + SLICES, ..), combined through lane swaps and LDS.  Bound by the latency of a
// thread's loads, four of each array in flight: at 193 tokens and V = 151936 four wavefronts per 64
// tokens walked 149 blocks each one by one in 73 us, with 32 slices 11 us.  Up to 64 vocabulary blocks
// 8 slices do (most of 32 would be empty, and their wavefronts keep other tokens out): us, 8 / 32
// slices, V = 1000 2500 tokens 3.1 / 4.0, 45000 4.5 / 7.5; V = 4096 45000 4.8 / 8.5; V = 10000 2500
// 4.0 / 4.7, 20000 4.7 / 7.0; V = 32000 257 6.0 / 5.4, 20000 7.3 / 9.1; V = 100000 2500 13.3 / 7.7.
//   rel == 0: psum = sum exp(z - pmax) per vocab block (log-prob only path)
//   rel == 1: psum = sum exp(z - s_t); with check != 0 a row whose max is too far from s_t
//             (exp(z - s_t) could leave float range) gets s_t = max and its token block is
//             marked for a second evaluation (whose partials loss_kernel merges).
constexpr int kMergeTok = 32;
template <int SLICES>
__global__ __launch_bounds__(32 * SLICES) void merge_kernel(
    const float* __restrict__ pmax, const float* __restrict__ psum,
    const float* __restrict__ psz, int64_t ldp, int32_t nmb, const float* __restrict__ zlab,
    const int32_t* __restrict__ yslab, int32_t Tc, int32_t rel, int32_t check,
    float* __restrict__ lse_out, float* __restrict__ logp_out, float* __restrict__ ent_out,
    float* __restrict__ shift, int32_t* __restrict__ redo_blk, int32_t* __restrict__ redo_count,
    int32_t* __restrict__ redo_any, int32_t block0) {
  constexpr int W = SLICES / 2;  // wavefronts
  __shared__ float sm[W][kMergeTok], ss[W][kMergeTok], sz[W][kMergeTok];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int tok = lane & 31, slice = wv * 2 + (lane >> 5);
  const int t = (block0 + int(blockIdx.x)) * kMergeTok + tok;
  const bool ok = t < Tc;
  const bool ent = psz != nullptr;
  // S = sum exp(z - ref), Z = sum exp(z - ref) z, both relative to the same reference
  float M = -INFINITY, S = 0.0f, Z = 0.0f;
  // one more partial (m, x, y) into (M, S, Z)
  auto add = [&](float m, float x, float y) {
    if (rel) {
      M = fmaxf(M, m);
      S += x;
      Z += y;
    } else if (m > M) {
      const float f = __expf(M - m);
      S = S * f + x;
      Z = Z * f + y;
      M = m;
    } else {
      const float f = __expf(m - M);
      S += x * f;
      Z += y * f;
    }
  };
  if (ok) {
    for (int b = slice; b < nmb; b += 4 * SLICES) {
      float m[4], x[4], y[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t o = int64_t(b + SLICES * u) * ldp + t;
        const bool in = b + SLICES * u < nmb;
        m[u] = in ? pmax[o] : 0.0f;
        x[u] = in ? psum[o] : 0.0f;
        y[u] = in && ent ? psz[o] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (b + SLICES * u < nmb) add(m[u], x[u], y[u]);
    }
  }
  // slices without a block hold (-inf, 0, 0) and add nothing
  auto join = [&](float m, float x, float y) {
    if (m > -INFINITY || x != 0.0f) add(m, x, y);
  };
  {
    const float m = __shfl_down(M, 32, 64), x = __shfl_down(S, 32, 64), y = __shfl_down(Z, 32, 64);
    join(m, x, y);
  }
  if (lane < 32) {
    sm[wv][tok] = M;
    ss[wv][tok] = S;
    sz[wv][tok] = Z;
  }
  __syncthreads();
  if (wv != 0 || lane >= 32 || !ok) return;
  M = sm[0][tok];
  S = ss[0][tok];
  Z = sz[0][tok];
#pragma unroll
  for (int w = 1; w < W; ++w) join(sm[w][tok], ss[w][tok], sz[w][tok]);
  const float s_t = (rel && shift) ? shift[t] : 0.0f;
  const float l = rel ? s_t + __logf(S) : M + __logf(S);
  const int y = yslab[t];
  if (lse_out) lse_out[t] = l;
  if (logp_out) logp_out[t] = y >= 0 ? zlab[t] - l : __int_as_float(0x7fc00000);
  // entropy -sum_v p_v log p_v = lse - sum_v p_v z_v, sum_v p_v z_v = Z / S
  if (ent_out) ent_out[t] = l - Z / S;
  if (rel && check && !(M - s_t < 60.0f && M - s_t > -60.0f)) {
    shift[t] = M;
    redo_blk[t / kBN] = 1;
    redo_any[0] = 1;
    atomicAdd(redo_count, 1);
  }
}

// sum over a block in a fixed order: wave butterflies, then the wave sums in order
constexpr int kSumThreads = 1024;
template <int THREADS = kSumThreads>
__device__ __forceinline__ double block_sum_d(double v, double* red) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wv] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) s += red[w];
  return s;
}

// sum of x[0..n) in float64, fixed order (one block): the mean entropy of the kept tokens
__global__ __launch_bounds__(kSumThreads) void sum_f32_kernel(const float* __restrict__ x, int64_t n,
                                                              float* __restrict__ out) {
  __shared__ double red[kSumThreads / 64];
  double s = 0.0;
#pragma unroll 4
  for (int64_t i = threadIdx.x; i < n; i += kSumThreads) s += double(x[i]);
  s = block_sum_d(s, red);
  if (threadIdx.x == 0) out[0] = float(s);
}

struct LossParams {
  float *logp, *lse, *ent;  // of all tokens (ent may be NULL)
  const float *old_logp, *ref_logp;
  const int32_t* row_index;
  const int64_t* seq_off;
  const float* adv;
  const int32_t* seq_index;
  int32_t S;
  int64_t T;
  int32_t seq_begin;        // of the slab
  int64_t row_base;
  int32_t algo, norm;
  float eps_low, eps_high, beta;
  const float* shift;       // NULL: no exp-logits, hence no shifts
  float* cslab;
  double* seq_loss;
  int32_t* seq_clip;
  int32_t* status;
  int32_t nadv;
  void* E1;                 // NULL without a backward
  int64_t ldE1;
  int32_t e_bf16;
  const int32_t* yslab;
  // the second evaluation's partials (rows with a shift)
  const float *psum, *psz, *zlab;
  int64_t ldp;
  int32_t nmb;
  const int32_t* redo_any;
  // the call's end
  const int32_t* redo_count;
  float *loss, *stats;
};

// sum of per-sequence loss terms in a fixed order (deterministic)
__global__ __launch_bounds__(kSumThreads) void loss_final_kernel(const LossParams p) {
  __shared__ double red[kSumThreads / 64];
  double s = 0.0, c = 0.0;
  // a contiguous chunk per thread keeps the order fixed for a given S
  const int per = (p.S + kSumThreads - 1) / kSumThreads;
  const int b = threadIdx.x * per, e = min(p.S, b + per);
  for (int i = b; i < e; ++i) {
    s += p.seq_loss[i];
    c += p.seq_clip[i];
  }
  s = block_sum_d(s, red);
  c = block_sum_d(c, red);
  if (threadIdx.x == 0) {
    p.loss[0] = float(s);
    if (p.stats) {
      p.stats[0] = float(c);
      p.stats[1] = float(p.redo_count[0]);
    }
  }
}

// sum of x[0], x[ld], .. x[(n - 1) ld] in order, 8 loads in flight.  (One after the other, the 594 of a
// row at V = 151936 took 0.2-0.4 ms of a loss call whose rows are all shifted: 588 tokens, d = 1536,
// 1519 us, 1330 so; 2048 tokens of one sequence, d = 3584, 7415 us, 7010 so.  16 gain 1% more there,
// but their code costs every call 0.5 us.)
__device__ __forceinline__ double column_sum_d(const float* x, int64_t ld, int n) {
  double s = 0.0;
  for (int m = 0; m < n; m += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = x[int64_t(min(m + u, n - 1)) * ld];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (m + u < n) s += double(v[u]);
  }
  return s;
}

// one block per sequence of the slab: g_t, c_t, the sequence's loss term and, with a backward,
// the one-hot term of each token folded into its exp-logit row (threads: launch_loss)
template <int THREADS>
__global__ __launch_bounds__(THREADS) void loss_kernel(const LossParams p) {
  __shared__ double red[THREADS / 64];
  const int i = p.seq_begin + blockIdx.x;
  const int64_t a = p.seq_off[i], b = p.seq_off[i + 1];
  const int64_t L = b - a;
  int ai = p.seq_index ? p.seq_index[i] : i;
  if (ai < 0 || ai >= p.nadv) {
    if (threadIdx.x == 0) set_status(p.status, FASTRL_SB_BAD_INDEX);
    ai = -1;
  }
  const double A = ai >= 0 ? double(p.adv[ai]) : 0.0;
  const double w = (p.norm == FASTRL_NORM_TOKEN_MEAN)
                       ? 1.0 / double(p.T)
                       : (L > 0 ? 1.0 / (double(p.S) * double(L)) : 0.0);
  const double lo = 1.0 - double(p.eps_low), hi = 1.0 + double(p.eps_high);
  const bool kl = p.beta != 0.0f;
  // rows that were evaluated again with a shift (rare): their log-sum-exp from the new partials,
  // by the thread that uses it below
  if (p.shift && L > 0 && p.redo_any[0] != 0) {
    for (int64_t t = a + threadIdx.x; t < b; t += THREADS) {
      const int64_t tl = t - p.row_base;
      const float s_t = p.shift[tl];
      if (s_t == 0.0f) continue;
      double S = 0.0, Z = 0.0;  // (one loop's code for both: it lies in every call's way)
#pragma clang loop unroll(disable)
      for (int k = p.psz ? 0 : 1; k < 2; ++k) {
        Z = S;
        S = column_sum_d((k == 0 ? p.psz : p.psum) + tl, p.ldp, p.nmb);
      }
      const float l = s_t + __logf(float(S));
      p.lse[t] = l;
      p.logp[t] = p.yslab[tl] >= 0 ? p.zlab[tl] - l : __int_as_float(0x7fc00000);
      if (p.ent) p.ent[t] = l - float(Z / S);
    }
  }
  double part = 0.0;  // this sequence's contribution to the loss
  int clip = 0;
  double sratio = 0.0, cseq = 0.0;
  if (p.algo == FASTRL_GSPO && L > 0) {
    double sl = 0.0;
    for (int64_t t = a + threadIdx.x; t < b; t += THREADS) {
      int64_t row = t;
      if (p.row_index) row = p.row_index[t];
      sl += double(p.logp[t]) - double(p.old_logp[row]);
    }
    sl = block_sum_d<THREADS>(sl, red);
    sratio = exp(sl / double(L));
    const double sur = fmin(sratio * A, fmin(fmax(sratio, lo), hi) * A);
    cseq = ((A >= 0.0 && sratio <= hi) || (A < 0.0 && sratio >= lo)) ? 1.0 : 0.0;
    if (threadIdx.x == 0) part = -(w * double(L)) * sur;
    clip = (cseq == 0.0) ? int(L) : 0;
  }
  double kpart = 0.0;
  for (int64_t t = a + threadIdx.x; t < b; t += THREADS) {
    int64_t row = t;
    if (p.row_index) row = p.row_index[t];
    const double x = p.logp[t];
    double g;
    if (p.algo == FASTRL_GSPO) {
      g = (w * double(L)) * (-cseq * sratio * A / double(L));
    } else {
      const double rho = exp(x - double(p.old_logp[row]));
      const double sur = fmin(rho * A, fmin(fmax(rho, lo), hi) * A);
      const double c = ((A >= 0.0 && rho <= hi) || (A < 0.0 && rho >= lo)) ? 1.0 : 0.0;
      kpart += -w * sur;
      g = w * (-c * rho * A);
      clip += (c == 0.0);
    }
    if (kl) {
      const double f = p.ref_logp[row];
      const double e = exp(f - x);
      kpart += double(p.beta) * w * (e - (f - x) - 1.0);
      g += double(p.beta) * w * (1.0 - e);
    }
    const int64_t tl = t - p.row_base;
    const float s_t = p.shift ? p.shift[tl] : 0.0f;
    p.cslab[tl] = float(g * exp(double(s_t) - double(p.lse[t])));
    // one-hot term of dZ folded into the exp-logits for the backward GEMMs: with
    // g_t = c_t exp(lse_t - s_t), c_t (E1[t][y_t] - exp(lse_t - s_t)) = c_t E1[t][y_t] - g_t
    const int y = p.E1 ? p.yslab[tl] : -1;
    if (y >= 0) {
      const double corr = exp(double(p.lse[t]) - double(s_t));
      const int64_t o = tl * p.ldE1 + y;
      if (p.e_bf16) {
        uint16_t* e = static_cast<uint16_t*>(p.E1) + o;
        *e = f32_to_bf16(float(double(bf16_to_f32(*e)) - corr));
      } else {
        float* e = static_cast<float*>(p.E1) + o;
        *e = float(double(*e) - corr);
      }
    }
  }
  kpart = block_sum_d<THREADS>(kpart, red);
  const double clips = block_sum_d<THREADS>(p.algo == FASTRL_GSPO ? 0.0 : double(clip), red);
  if (threadIdx.x == 0) {
    p.seq_loss[i] = part + kpart;
    p.seq_clip[i] = p.algo == FASTRL_GSPO ? clip : int(clips);
  }
}

// out[c][r] = scale(r) * in[row(r)][c], zero for r in [R, Rpad): 64 x 64 tiles through LDS with
// 16-byte global loads and stores (C is a multiple of 8, in 16-byte aligned, Rpad and ldo
// multiples of 64, out 256-byte aligned)
__global__ __launch_bounds__(256) void transpose_scale_kernel(
    const uint16_t* __restrict__ in, const int32_t* __restrict__ row_index, int64_t row_base,
    int32_t R, int32_t Rpad, int32_t C, const float* __restrict__ scale, uint16_t* __restrict__ out,
    int64_t ldo) {
  constexpr int VEC = 8;          // elements per 16-byte piece
  constexpr int LPR = 64 / VEC;   // threads per 64-element tile row
  constexpr int RPP = 256 / LPR;  // tile rows per pass
  __shared__ float tile[64][65];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const int tid = threadIdx.x;
  const int l = (tid % LPR) * VEC;
  for (int rr = tid / LPR; rr < 64; rr += RPP) {
    const int r = r0 + rr;
    float v[VEC];
    if (r < R && c0 + l < C) {
      int64_t row = row_base + r;
      if (row_index) row = row_index[row];
      const u32x4_t raw = *reinterpret_cast<const u32x4_t*>(in + row * C + c0 + l);
      const float sc = scale ? scale[r] : 1.0f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v[2 * q] = bf16_to_f32(uint16_t(raw[q] & 0xffffu)) * sc;
        v[2 * q + 1] = bf16_to_f32(uint16_t(raw[q] >> 16)) * sc;
      }
    } else {
#pragma unroll
      for (int q = 0; q < VEC; ++q) v[q] = 0.0f;
    }
#pragma unroll
    for (int q = 0; q < VEC; ++q) tile[rr][l + q] = v[q];
  }
  __syncthreads();
  for (int cc = tid / LPR; cc < 64; cc += RPP) {
    const int c = c0 + cc;
    if (c < C && r0 + l < Rpad) {
      u32x4_t o;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        o[q] = uint32_t(f32_to_bf16(tile[l + 2 * q][cc])) |
               (uint32_t(f32_to_bf16(tile[l + 2 * q + 1][cc])) << 16);
      *reinterpret_cast<u32x4_t*>(out + int64_t(c) * ldo + r0 + l) = o;
    }
  }
}

// out[r] = scale[r] * in[row(r)] for r < R, zero rows up to Rpad (float32 dW: hidden rows times c_t)
__global__ __launch_bounds__(256) void scale_rows_f32_kernel(
    const float* __restrict__ in, const int32_t* __restrict__ row_index, int64_t row_base,
    int32_t R, int32_t Rpad, int32_t C, const float* __restrict__ scale, float* __restrict__ out) {
  const int c4 = C / 4;
  const int64_t n4 = int64_t(Rpad) * c4;
  // (once around, unless a launch cannot hold a thread for each piece)
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n4; i += int64_t(gridDim.x) * 256) {
    const int r = int(i / c4);
    f32x4_t v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (r < R) {
      int64_t row = row_base + r;
      if (row_index) row = row_index[row];
      v = reinterpret_cast<const f32x4_t*>(in + row * C)[i % c4];
      const float s = scale[r];
      v = f32x4_t{s * v[0], s * v[1], s * v[2], s * v[3]};
    }
    reinterpret_cast<f32x4_t*>(out)[i] = v;
  }
}

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x)
    p[i] = v;
}

// ------------------------------------------------------------------ host side

static inline int64_t rup(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

constexpr int kMaxKSplit = 32;  // parts of K of a dhidden GEMM
constexpr int BK_F32 = 32;      // K step of the float32 GEMMs
// blocks of one launch at most: a launch's threads number below 2^32, and the largest blocks are of 1024
constexpr int64_t kMaxBlocks = int64_t(1) << 21;

static int launch_dh_reduce(const GemmParams& q, hipStream_t stream) {
  const int64_t n4 = int64_t(q.M) * (q.d / 4);
  hipLaunchKernelGGL(dh_reduce_kernel, dim3(unsigned((n4 + 255) / 256)), dim3(256), 0, stream,
                     q.part, q.ksplit, q.M, q.d, q.cslab, q.dH, q.dH_bf16);
  FR_LAUNCHED();
  return FASTRL_OK;
}

// Tile group of a GEMM (tile_coords), measured back to back on the two hidden sizes of the
// workloads: the logits GEMM takes 32 at K = d = 3584 (8 loses 4%, 16 1%; 64 is level) and, with
// exp-logits stored, 16 at d = 1536 (32 loses 2% on that GEMM, 64 3%); without them 32 there too
// (18900 tokens: 6356 us against 6519 with 16 and 6741 with 8).  dhidden 4 when d spans 14 column
// blocks and 8 when it spans 6, the dW tiles 4 (2 to 16 within 0.7% of each other).
static int tile_group(int mode, int32_t K, int32_t nnb, bool store_e = false) {
  if (mode == MODE_FWD) return K <= 2048 && store_e ? 16 : 32;
  if (mode == MODE_DH) return nnb <= 8 ? 8 : 4;
  return 4;
}

// Rows of the bf16 GEMMs' row-by-row operands from which lm_wide_kernel runs, in elements: a lane's
// offset inside 8 rows is 32 bits of bytes elsewhere (a row of this length is half a GiB; K-major
// operands have no such limit)
constexpr int64_t kMaxLd = int64_t(1) << 28;

template <int MODE>
static bool wide_rows(const GemmParams& p) {
  return p.lda >= kMaxLd || (MODE == MODE_DH && p.ldb >= kMaxLd);
}

template <int MODE>
static int launch_wide(GemmParams p, int kind, double flops, hipStream_t stream) {
  p.nmb = int((p.M + kBM - 1) / kBM);
  p.nnb = int((p.N + kBN - 1) / kBN);
  p.group = tile_group(MODE == MODE_DHT ? int(MODE_DH) : MODE, p.K, p.nnb, p.store_e != 0);
  p.narrow = p.tail = 0;
  const int64_t nblk = int64_t(p.nmb) * p.nnb;
  if (nblk == 0) return FASTRL_OK;
  FR_CHECK_ARG(MODE == MODE_FWD || p.K % 64 == 0, FASTRL_ERR_UNSUPPORTED, "GEMM: unsupported shape");
  ProfScope prof(kind, stream, flops);
  hipLaunchKernelGGL(lm_wide_kernel<MODE>, dim3(unsigned(nblk)), dim3(kThreads), 0, stream, p);
  FR_LAUNCHED();
  return FASTRL_OK;
}

// Tiles of a logits GEMM; returns the blocks.  The last N % 256 tokens take a column of narrow tiles
// (64, 128 or 192 wide) in place of whole ones that are mostly padding.  Without those, a last
// wave of at most 128 (64) whole tiles on the 256 compute units is cut into 2 (4) pieces per tile,
// which run at once.  token_logprob, us, whole tiles only -> so: d = 1536 (V = 151936) 16 tokens
// 141 -> 104, 193 145 -> 137, 300 215 -> 174, 1200 488 -> 473; d = 3584 (V = 152064) 16 284 -> 210, 300
// 442 -> 369, 2309 1997 -> 1927, 33733 level.
static int64_t fwd_tiles(GemmParams& p) {
  p.nmb = int((p.M + kBM - 1) / kBM);
  p.nnb = int((p.N + kBN - 1) / kBN);
  p.narrow = ((p.N % kBN + 63) / 64) % 4;
  p.group = tile_group(MODE_FWD, p.K, p.nnb, p.store_e != 0);
  const int64_t whole = int64_t(p.nmb) * p.nnb;
  const int last = int(whole % 256);
  p.tail = p.narrow == 0 && last <= 128 && whole < kMaxBlocks ? last : 0;
  p.pieces = p.tail == 0 ? 1 : p.tail <= 64 ? 4 : 2;
  return whole + int64_t(p.tail) * (p.pieces - 1);
}

// Tiles of a float32 GEMM.  The gradient GEMMs take 128 x 128 tiles where those alone fill the
// chip twice, else 64 x 64; dhidden then cuts its K (the vocabulary) so that there are about two
// blocks per compute unit, of at least 8 K steps each.
template <int MODE, int BM, int BN, int WM, int WN, int ST>
static int launch_f32_tiles(GemmParams p, int kind, double flops, hipStream_t stream) {
  p.nmb = int((p.M + BM - 1) / BM);
  p.nnb = int((p.N + BN - 1) / BN);
  p.group = 8;
  const int64_t nblk = int64_t(p.nmb) * p.nnb * (MODE == MODE_DH ? p.ksplit : 1);
  if (nblk == 0) return FASTRL_OK;
  FR_CHECK_ARG(nblk < (int64_t(1) << 31) && p.K >= 8 && p.N >= (MODE == MODE_FWD ? 1 : 8) &&
                   (MODE == MODE_FWD ? p.K % 8 == 0 : p.K % BK_F32 == 0),
               FASTRL_ERR_UNSUPPORTED, "float32 GEMM: unsupported shape");
  {
    ProfScope prof(kind, stream, flops);
    for (int64_t b = 0; b < nblk; b += kMaxBlocks) {
      p.block0 = int32_t(b);
      hipLaunchKernelGGL((f32_gemm_kernel<MODE, BM, BN, WM, WN, ST>),
                         dim3(unsigned(std::min(nblk - b, kMaxBlocks))), dim3(64 * WM * WN), 0, stream,
                         p);
      FR_LAUNCHED();
    }
  }
  if (MODE == MODE_DH && p.ksplit > 1) return launch_dh_reduce(p, stream);
  return FASTRL_OK;
}

static bool f32_big_tiles(int64_t M, int64_t N) {
  return ((M + 127) / 128) * ((N + 127) / 128) >= 512;
}

static int f32_ksplit(int64_t M, int64_t N, int32_t V) {
  const int64_t b = f32_big_tiles(M, N) ? 128 : 64;
  const int64_t nt = ((M + b - 1) / b) * ((N + b - 1) / b), nk = (V + BK_F32 - 1) / BK_F32;
  return int(std::max<int64_t>(1, std::min<int64_t>({512 / nt, nk / 8, kMaxKSplit})));
}

template <int MODE>
static int launch_f32(const GemmParams& p, int kind, double flops, hipStream_t stream) {
  if constexpr (MODE == MODE_FWD)
    return launch_f32_tiles<MODE, 256, 64, 4, 2, 2>(p, kind, flops, stream);
  else if (f32_big_tiles(p.M, p.N))
    return launch_f32_tiles<MODE, 128, 128, 2, 2, 2>(p, kind, flops, stream);
  else
    return launch_f32_tiles<MODE, 64, 64, 2, 2, 4>(p, kind, flops, stream);
}

template <typename T, int MODE>
static int launch_gemm(GemmParams p, int kind, double flops, hipStream_t stream) {
  if constexpr (sizeof(T) == 4) return launch_f32<MODE>(p, kind, flops, stream);
  else {
  if (wide_rows<MODE>(p)) return launch_wide<MODE>(p, kind, flops, stream);
  int64_t nblk;
  if constexpr (MODE == MODE_FWD) {
    nblk = fwd_tiles(p);
  } else {
    p.nmb = int((p.M + kBM - 1) / kBM);
    p.nnb = int((p.N + kBN - 1) / kBN);
    p.group = tile_group(MODE, p.K, p.nnb);
    nblk = int64_t(p.nmb) * p.nnb;
  }
  if (nblk == 0) return FASTRL_OK;
  // transposed dW: whole 64-k tiles, whole 256-column tiles of the K-major E, 16-byte dW rows
  FR_CHECK_ARG(MODE != MODE_DWT || (p.K % 64 == 0 && p.ldb >= int64_t(p.nnb) * kBN &&
                                    p.ldb % 8 == 0 && p.d % 4 == 0 && p.M == p.d),
               FASTRL_ERR_UNSUPPORTED, "transposed dW GEMM: unsupported shape");
  ProfScope prof(kind, stream, flops);
  hipLaunchKernelGGL((lm_gemm_kernel<T, MODE>), dim3(unsigned(nblk)), dim3(kThreads), 0, stream, p);
  FR_LAUNCHED();
  return FASTRL_OK;
  }
}

// dhidden (q, MODE_DH) and transposed dW (r, MODE_DWT) of one bf16 slab in one launch
static int launch_bwd(GemmParams q, GemmParams r, double flops, hipStream_t stream) {
  q.nmb = int((q.M + kBM - 1) / kBM);
  q.nnb = int((q.N + kBN - 1) / kBN);
  r.nmb = int((r.M + kBM - 1) / kBM);
  r.nnb = int((r.N + kBN - 1) / kBN);
  q.group = tile_group(MODE_DH, q.K, q.nnb);
  r.group = tile_group(MODE_DWT, r.K, r.nnb);
  const int64_t nh = int64_t(q.nmb) * q.nnb, nw = int64_t(r.nmb) * r.nnb;
  if (nh + nw == 0) return FASTRL_OK;
  FR_CHECK_ARG(nh + nw < (int64_t(1) << 31), FASTRL_ERR_UNSUPPORTED, "backward GEMMs: grid too large");
  FR_CHECK_ARG(r.K % 64 == 0 && r.ldb >= int64_t(r.nnb) * kBN && r.ldb % 8 == 0 && r.d % 4 == 0 &&
                   r.M == r.d,
               FASTRL_ERR_UNSUPPORTED, "transposed dW GEMM: unsupported shape");
  ProfScope prof(FASTRL_K_BACKWARD, stream, flops);
  hipLaunchKernelGGL(lm_bwd_kernel, dim3(unsigned(nh + nw)), dim3(512), 0, stream, q, r);
  FR_LAUNCHED();
  return FASTRL_OK;
}

// Calls of few tokens read W itself in dhidden (MODE_DHT): the transposed copy of W, built per call
// (0.39 ms at 7B, 0.16 ms at d = 1536), costs more there than the transposing LDS reads do, and K can
// be cut.  Beside dW tiles, whose traffic slows those reads, up to kDirectTokens tokens; dhidden alone
// up to kDirectTokensAlone.  Measured, transposed copy / W itself, us a call: both gradients,
// d = 1536 (V = 151936) 1024 tokens 3608 / 1364, 2048 4083 / 2407, 4096 5068 / 4634, 6144 6744 / 6816,
// 8192 8788 / 8863, 16384 17221 / 17701; d = 3584 (V = 152064) 2048 5717 / 5364, 4096 10043 / 9970,
// 8192 19672 / 19735, 16384 39265 / 39623, 20480 49089 / 50019, 32768 76808 / 80305; d = 896
// (V = 151936) 4096 4190 / 3138, 8192 5990 / 5992, 16384 11704 / 11989; d = 2048 (V = 100000) 4096
// 3948 / 3899, 8192 7569 / 7626, 16384 14880 / 15244.  dhidden alone, d = 1536 8192 6313 / 6171, 16384
// 12803 / 12167, 32768 23672 / 24838; d = 3584 8192 13275 / 13357, 16384 27377 / 26917, 32768 52193 /
// 54763.
constexpr int64_t kDirectTokens = 6144, kDirectTokensAlone = 20480;

// (float32 dhidden always reads W itself)
static bool direct_dh(const fastrl_loss_args& a) {
  return a.dhidden != nullptr &&
         (a.dtype == FASTRL_F32 || a.T <= (a.dW ? kDirectTokens : kDirectTokensAlone));
}

// Parts of K for the dhidden tiles of a Tc-token slab: the count whose estimated time is least,
// in K steps of 64 (~1.2 us each on a compute unit of its own).  The launch lasts at least as
// long as its dhidden rounds (parts x tiles over 256 compute units, each K / parts plus ~8 steps
// of start and end) and as its total work spread evenly (a dW tile: its K plus ~12 steps, mostly
// dW's own traffic); parts add their float32 sums' traffic (written and read at ~5 TB/s).  Next to
// dW tiles K stays whole where a tile's chain is hidden behind the rest, else the parts are a power
// of two (with 15% on their rounds, which the dW tiles beside them slow down), and from 4 on blocks take the parts of a tile in a row: blocks are dealt round-robin to the
// 8 XCDs, so an XCD sees only one or two parts and its L2 holds their strips (2% assumed).
// Measured, us a call (1, 2, 4, 8, 16 parts; the rule's choice in brackets): d = 1536, V = 151936,
// 588 tokens 3234, 1876, 1212, [1005], 1006; 2048 tokens 4090, 2676, [2398], 2441, 2532; 8192
// [8814], 8900, 9004, 9474, 9690; d = 3584, V = 152064, 1000 tokens 4290, 2988, [2913], 2929, 3007;
// 1975 tokens [5068], .., 5141; 8192 [19622], 19838, 19984, 21080, 21651.
static int dh_ksplit(int32_t Tc, int32_t d, int32_t V, int32_t dtype, bool dw) {
  if (dtype == FASTRL_F32) return f32_ksplit(Tc, d, V);
  if (rup(V, kBM) >= kMaxLd) return 1;  // lm_wide_kernel
  const double nt = double((Tc + kBM - 1) / kBM) * double((d + kBN - 1) / kBN);
  const double nk = double((V + 63) / 64);
  const double wt = dw ? double((V + kBN - 1) / kBN) * double((d + kBM - 1) / kBM) : 0.0;
  const double wk = double((Tc + 63) / 64) + 12.0;
  int best = 1;
  double best_t = 0.0;
  for (int s = 1; s <= kMaxKSplit && double(s) * 8.0 <= nk; s += dw ? s : 1) {
    const double part = nk / s + 8.0;
    const double rounds = std::ceil(nt * s / 256.0) * part;
    const double even = (nt * s * part + wt * wk) / 256.0 + (dw ? wk : 0.0);
    if (dw && s == 1 && rounds <= even) return 1;
    double t = std::max(dw ? 1.15 * rounds : rounds, even);
    if (s > 1) t += double(s) * Tc * d * 8.0 / 5e12 / 1.2e-6;
    if (dw && s >= 4) t *= 0.98;
    if (s == 1 || t < best_t) {
      best = s;
      best_t = t;
    }
  }
  return best;
}

static int launch_bwd_direct(GemmParams q, GemmParams r, bool dw, double flops,
                             hipStream_t stream) {
  q.nmb = int((q.M + kBM - 1) / kBM);
  q.nnb = int((q.N + kBN - 1) / kBN);
  r.nmb = dw ? int((r.M + kBM - 1) / kBM) : 0;
  r.nnb = dw ? int((r.N + kBN - 1) / kBN) : 0;
  q.group = tile_group(MODE_DH, q.K, q.nnb);
  q.part_first = dw && q.ksplit >= 4;
  r.group = tile_group(MODE_DWT, r.K, r.nnb);
  const int64_t nh = int64_t(q.nmb) * q.nnb * q.ksplit, nw = int64_t(r.nmb) * r.nnb;
  if (nh + nw == 0) return FASTRL_OK;
  FR_CHECK_ARG(nh + nw < (int64_t(1) << 31), FASTRL_ERR_UNSUPPORTED, "backward GEMMs: grid too large");
  FR_CHECK_ARG(q.K % 64 == 0 && q.K <= q.lda && q.ldb % 8 == 0 && q.N >= 8 && q.ksplit >= 1 &&
                   q.ksplit * 64 <= q.K && (q.ksplit == 1 || q.part),
               FASTRL_ERR_UNSUPPORTED, "direct dhidden GEMM: unsupported shape");
  FR_CHECK_ARG(!dw || (r.K % 64 == 0 && r.ldb >= int64_t(r.nnb) * kBN && r.ldb % 8 == 0 &&
                       r.d % 4 == 0 && r.M == r.d),
               FASTRL_ERR_UNSUPPORTED, "transposed dW GEMM: unsupported shape");
  {
    ProfScope prof(dw ? FASTRL_K_BACKWARD : FASTRL_K_DHIDDEN, stream, flops);
    hipLaunchKernelGGL(lm_bwd_direct_kernel, dim3(unsigned(nh + nw)), dim3(512), 0, stream, q, r);
    FR_LAUNCHED();
  }
  if (q.ksplit > 1) return launch_dh_reduce(q, stream);
  return FASTRL_OK;
}

// the second evaluation of marked token blocks (store_e == 2): bf16 through lm_redo_kernel
template <typename T>
static int launch_redo(GemmParams p, hipStream_t stream) {
  p.store_e = 2;
  if constexpr (sizeof(T) != 2) return launch_gemm<T, MODE_FWD>(p, -1, 0.0, stream);
  if (wide_rows<MODE_FWD>(p)) return launch_wide<MODE_FWD>(p, -1, 0.0, stream);
  p.nmb = int((p.M + kBM - 1) / kBM);
  p.nnb = int((p.N + kBN - 1) / kBN);
  p.group = tile_group(MODE_FWD, p.K, p.nnb, true);
  const int64_t nblk = int64_t(p.nmb) * p.nnb;
  if (nblk == 0) return FASTRL_OK;
  hipLaunchKernelGGL(lm_redo_kernel, dim3(unsigned(std::min<int64_t>(nblk, 256))), dim3(512), 0,
                     stream, p);
  FR_LAUNCHED();
  return FASTRL_OK;
}

#define FR_TRY(x)                 \
  do {                            \
    int rc_ = (x);                \
    if (rc_ != FASTRL_OK) return rc_; \
  } while (0)

static inline unsigned nb1d(int64_t n, int b) { return unsigned((n + b - 1) / b); }

// partials -> lse, logp (and entropy); rel: of stored exp-logits, whose rows are checked for a shift
static int launch_merge(const float* pmax, const float* psum, const float* psz, int64_t ldp,
                        int32_t nmb, const float* zlab, const int32_t* yslab, int32_t Tc, bool rel,
                        float* lse, float* logp, float* ent, float* shift, int32_t* redo_blk,
                        int32_t* redo_count, int32_t* redo_any, hipStream_t stream) {
  const int64_t blocks = nb1d(Tc, kMergeTok);
  const bool few = nmb <= 64;
  for (int64_t b = 0; b < blocks; b += kMaxBlocks) {
    hipLaunchKernelGGL(few ? merge_kernel<8> : merge_kernel<32>,
                       dim3(unsigned(std::min(blocks - b, kMaxBlocks))), dim3(few ? 256 : 1024), 0,
                       stream, pmax, psum, psz, ldp, nmb, zlab, yslab, Tc, rel ? 1 : 0, rel ? 1 : 0,
                       lse, logp, ent, shift, redo_blk, redo_count, redo_any, int32_t(b));
    FR_LAUNCHED();
  }
  return FASTRL_OK;
}

// The loss kernel over a slab's n sequences of Tc tokens, the longest of `longest`: 256 threads a
// sequence up to 512 tokens, and where there are many and most are shorter; 1024 for the latency of a
// few long ones.  Loss kernel, us, 256 / 1024 threads: 3333 sequences of 6 tokens 10.4 / 44.0, 1000 of
// 30 4.9 / 14.6, 60 of 500 4.7 / 5.0, 16 of 500 5.0 / 5.1, 8 of 1000 7.2 / 5.7, 20 of 1500 8.2 / 6.0,
// one of 16384 53.8 / 23.2.
static int launch_loss(const LossParams& lp, int32_t n, int64_t Tc, int64_t longest,
                       hipStream_t stream) {
  const bool few = longest <= 512 || (n >= 512 && Tc <= 256 * int64_t(n));
  hipLaunchKernelGGL(few ? loss_kernel<256> : loss_kernel<kSumThreads>, dim3(unsigned(n)),
                     dim3(few ? 256 : kSumThreads), 0, stream, lp);
  FR_LAUNCHED();
  return FASTRL_OK;
}

// ---------------------------------------------------------------- token log-prob only
constexpr int64_t kLogprobChunk = 65536;

struct LogprobWs {
  float *pmax, *psum, *zlab;
  int32_t* yslab;
};

// tokens per chunk for T tokens when at most `chunk` fit (a multiple of 256)
static int64_t logprob_chunk(int64_t T, int64_t chunk) {
  return rup(std::min<int64_t>(std::max<int64_t>(T, 1), chunk), 256);
}

static size_t carve_logprob(Carver& c, LogprobWs& w, int64_t ch, int32_t V) {
  const int64_t nmb = (V + kBM - 1) / kBM;
  w.pmax = c.take<float>(size_t(nmb * ch));
  w.psum = c.take<float>(size_t(nmb * ch));
  w.zlab = c.take<float>(size_t(ch));
  w.yslab = c.take<int32_t>(size_t(ch));
  return c.size();
}

size_t token_logprob_workspace(int64_t T, int32_t d, int32_t V, int32_t dtype) {
  (void)d;
  (void)dtype;
  Carver c(nullptr);
  LogprobWs w;
  return carve_logprob(c, w, logprob_chunk(T, kLogprobChunk), V);
}

// Chunks of at most `chunk` tokens through the logits GEMM (partials only) and the merge;
// every token's result depends on its own logits alone, so the chunking changes nothing.
// prof: record the GEMM launches in the kernel-timing recorder.
template <typename T>
static int token_logprob_impl(const void* hidden, const int32_t* row_index, const void* W,
                              int64_t Tn, int32_t d, int32_t V, const int32_t* token_ids,
                              float* logp, float* lse, int32_t* status, void* ws,
                              int64_t chunk, bool prof, hipStream_t stream) {
  Carver c(ws);
  LogprobWs w;
  const int64_t ch = logprob_chunk(Tn, chunk);
  carve_logprob(c, w, ch, V);
  for (int64_t t0 = 0; t0 < Tn; t0 += ch) {
    const int32_t Tc = int32_t(std::min<int64_t>(ch, Tn - t0));
    hipLaunchKernelGGL(slab_prep_kernel, dim3(nb1d(Tc, 256)), dim3(256), 0, stream, token_ids,
                       row_index, t0, Tc, V, w.yslab, (float*)nullptr, status,
                       (int32_t*)nullptr, 0, (int32_t*)nullptr);
    FR_LAUNCHED();
    GemmParams p{};
    p.A = W; p.lda = d; p.M = V;
    p.B = hidden; p.ldb = d; p.N = Tc; p.b_rows = row_index; p.b_row_base = t0;
    p.K = d;
    p.pmax = w.pmax; p.psum = w.psum; p.ldp = ch; p.zlab = w.zlab; p.yslab = w.yslab;
    p.Vreal = V; p.store_e = 0;
    FR_TRY((launch_gemm<T, MODE_FWD>(p, prof ? FASTRL_K_LOGITS_FWD : -1,
                                     2.0 * V * double(Tc) * d, stream)));
    const int32_t nmb = (V + kBM - 1) / kBM;
    FR_TRY(launch_merge(w.pmax, w.psum, nullptr, ch, nmb, w.zlab, w.yslab, Tc, false,
                        lse ? lse + t0 : nullptr, logp + t0, nullptr, nullptr, nullptr, nullptr,
                        nullptr, stream));
  }
  return FASTRL_OK;
}

int run_token_logprob(const void* hidden, const int32_t* row_index, const void* W,
                      int32_t dtype, int64_t T, int32_t d, int32_t V,
                      const int32_t* token_ids, float* logp, float* lse, int32_t* status,
                      void* ws, hipStream_t stream) {
  if (dtype == FASTRL_BF16)
    return token_logprob_impl<uint16_t>(hidden, row_index, W, T, d, V, token_ids, logp, lse,
                                        status, ws, kLogprobChunk, true, stream);
  return token_logprob_impl<float>(hidden, row_index, W, T, d, V, token_ids, logp, lse, status,
                                   ws, kLogprobChunk, true, stream);
}

// ---- the allocation-free variant: its scratch is a fixed device array --------------------
// kNoAllocScratchBytes of device memory per GPU, held from the library's first use on that
// GPU until the process ends.  In host code `scratch` names a host-side stand-in, not the
// device copy: its device address is fetched once per device (hipGetSymbolAddress, with that
// device current) and only that address reaches kernels.  Every call on a GPU shares that
// GPU's array, so calls that overlap on one GPU (two streams, two threads) race.  Nothing in
// it has to start at zero: each chunk writes every partial, label and logit it reads.
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;
static __device__ __align__(256) char scratch[kNoAllocScratchBytes];

constexpr int kMaxScratchDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_dev[kMaxScratchDevices] = {};

size_t token_logprob_noalloc_scratch_bytes() { return kNoAllocScratchBytes; }

// the most tokens per chunk (a multiple of 256) whose partials fit in the scratch; 0 if not
// even 256 do
int64_t token_logprob_noalloc_chunk(int32_t V) {
  int64_t lo = 0;
  for (int64_t ch = 256; ch <= kLogprobChunk; ch += 256) {
    Carver c(nullptr);
    LogprobWs w;
    if (carve_logprob(c, w, ch, V) > kNoAllocScratchBytes) break;
    lo = ch;
  }
  return lo;
}

int run_token_logprob_noalloc(const void* hidden, const int32_t* row_index, const void* W,
                              int32_t dtype, int64_t T, int32_t d, int32_t V,
                              const int32_t* token_ids, float* logp, float* lse,
                              int32_t* status, hipStream_t stream) {
  const int64_t chunk = token_logprob_noalloc_chunk(V);
  FR_CHECK_ARG(chunk >= 256, FASTRL_ERR_SHAPE,
               "fastrl_token_logprob_noalloc: V = " + std::to_string(V) +
                   " needs more than the fixed scratch of " +
                   std::to_string(kNoAllocScratchBytes >> 20) + " MiB for 256 tokens");
  int dev = -1;
  FR_HIP(hipGetDevice(&dev));
  FR_CHECK_ARG(dev >= 0 && dev < kMaxScratchDevices, FASTRL_ERR_UNSUPPORTED,
               "fastrl_token_logprob_noalloc: device ordinal out of range");
  if (stream) {
    int sdev = -1;
    FR_HIP(hipStreamGetDevice(stream, &sdev));
    FR_CHECK_ARG(sdev == dev, FASTRL_ERR_VALUE,
                 "fastrl_token_logprob_noalloc: the stream belongs to another device than the "
                 "current one");
  }
  void* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
      void* p = nullptr;
      FR_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
      FR_CHECK_ARG(p != nullptr, FASTRL_ERR_HIP,
                   "fastrl_token_logprob_noalloc: no device address for the scratch array");
      g_scratch_dev[dev] = p;
    }
    ptr = g_scratch_dev[dev];
  }
  if (T == 0) return FASTRL_OK;
  if (dtype == FASTRL_BF16)
    return token_logprob_impl<uint16_t>(hidden, row_index, W, T, d, V, token_ids, logp, lse,
                                        status, ptr, chunk, false, stream);
  return token_logprob_impl<float>(hidden, row_index, W, T, d, V, token_ids, logp, lse, status,
                                   ptr, chunk, false, stream);
}

// ---------------------------------------------------------------- loss forward/backward
// Default slab: 32768 tokens whatever T is, so the exp-logit buffer [slab, V_pad] is bounded
// (10 GB in bf16 at V = 152064) and no [T, V] array exists for any T; a caller picks another
// bound with slab_tokens.
constexpr int64_t kDefaultSlabTokens = 32768;

struct SlabPlan {
  std::vector<int32_t> seq_begin;  // first sequence of each slab; back() == S
  int64_t tc_max = 0;
};

// Whole sequences per slab.  Each slab takes an even share of what is left, counted afresh
// after every slab (ceil(remaining / cap) slabs to go, so the shares stay close to cap): it
// ends at the sequence boundary closest to that share, never past 1.25 cap unless a single
// sequence is longer, so every slab holds at most max(1.25 cap, longest sequence) tokens.
// A slab holds at least one token while any are left (empty sequences join the slab of
// their neighbours); only T == 0 gives a slab without tokens.
static SlabPlan plan_slabs(const int64_t* off, int32_t S, int64_t cap) {
  SlabPlan pl;
  const int64_t hard = cap + cap / 4;
  int32_t i = 0;
  while (i < S) {
    pl.seq_begin.push_back(i);
    const int64_t start = off[i];
    const int64_t rem = off[S] - start;
    const int64_t left = std::max<int64_t>(1, (rem + cap - 1) / cap);
    int32_t best = S;
    if (left > 1) {
      const int64_t target = (rem + left - 1) / left;
      best = i + 1;
      while (best < S && off[best] == start) ++best;  // at least one token
      for (int32_t j = best + 1; j <= S && off[j] - start <= hard; ++j)
        if (std::llabs(off[j] - start - target) < std::llabs(off[best] - start - target)) best = j;
      while (best < S && off[best + 1] == off[best]) ++best;  // trailing empty sequences
    }
    pl.tc_max = std::max<int64_t>(pl.tc_max, off[best] - start);
    i = best;
  }
  pl.seq_begin.push_back(S);
  return pl;
}

struct LossWs {
  void *WT, *E1, *Bd;
  float *pmax, *psum, *psz, *ent, *zlab, *shift, *cslab, *lse, *logp;
  int32_t *yslab, *redo_blk, *redo_count, *seq_clip;
  double* seq_loss;
};

static size_t carve_loss(Carver& c, LossWs& w, const fastrl_loss_args& a, const SlabPlan& pl) {
  const int64_t tc_max = pl.tc_max;
  const int esz = a.dtype == FASTRL_BF16 ? 2 : 4;
  const int64_t Vpad = rup(a.V, kBM);
  const int64_t tcp = rup(std::max<int64_t>(tc_max, 1), kBN);
  const int64_t nmb = Vpad / kBM;
  const bool dh = a.dhidden != nullptr, dw = a.dW != nullptr;
  // one region holds W^T or, where dhidden reads W itself, its float32 parts (bf16: room for W^T in
  // both cases, the size that callers know; float32 never transposes W)
  int64_t wt = dh && a.dtype == FASTRL_BF16 ? int64_t(a.d) * Vpad * 2 : 0;
  if (direct_dh(a))
    for (size_t si = 0; si + 1 < pl.seq_begin.size(); ++si) {
      const int64_t Tc = a.seq_off_host[pl.seq_begin[si + 1]] - a.seq_off_host[pl.seq_begin[si]];
      const int ks = Tc > 0 ? dh_ksplit(int32_t(Tc), a.d, a.V, a.dtype, dw) : 1;
      if (ks > 1) wt = std::max(wt, Tc * ks * a.d * int64_t(sizeof(float)));
    }
  w.WT = wt > 0 ? c.take<char>(size_t(wt)) : nullptr;
  w.E1 = (dh || dw) ? c.take<char>(size_t(tcp) * Vpad * esz) : nullptr;
  w.Bd = dw ? c.take<char>(size_t(a.d) * tcp * esz) : nullptr;
  w.pmax = c.take<float>(size_t(nmb * tcp));
  w.psum = c.take<float>(size_t(nmb * tcp));
  const bool ent = a.entropy != nullptr || a.entropy_sum != nullptr;
  w.psz = ent ? c.take<float>(size_t(nmb * tcp)) : nullptr;
  w.ent = a.entropy ? a.entropy
                    : (a.entropy_sum ? c.take<float>(size_t(std::max<int64_t>(a.T, 1))) : nullptr);
  w.zlab = c.take<float>(size_t(tcp));
  w.shift = c.take<float>(size_t(tcp));
  w.cslab = c.take<float>(size_t(tcp));
  w.yslab = c.take<int32_t>(size_t(tcp));
  w.redo_blk = c.take<int32_t>(size_t(tcp / kBN + 1));  // + the slab's any-marked flag
  w.redo_count = c.take<int32_t>(1);
  w.lse = a.lse ? a.lse : c.take<float>(size_t(std::max<int64_t>(a.T, 1)));
  w.logp = a.logp ? a.logp : c.take<float>(size_t(std::max<int64_t>(a.T, 1)));
  w.seq_loss = c.take<double>(size_t(std::max(a.S, 1)));
  w.seq_clip = c.take<int32_t>(size_t(std::max(a.S, 1)));
  return c.size();
}

static int64_t slab_cap(const fastrl_loss_args& a) {
  return a.slab_tokens > 0 ? a.slab_tokens : kDefaultSlabTokens;
}

int policy_loss_slab_plan(const fastrl_loss_args& a, int32_t* seq_begin, int32_t capacity,
                          int64_t* tc_max) {
  SlabPlan pl = plan_slabs(a.seq_off_host, a.S, slab_cap(a));
  const int32_t n = int32_t(pl.seq_begin.size()) - 1;
  if (tc_max) *tc_max = pl.tc_max;
  if (seq_begin && capacity > n)
    for (int32_t k = 0; k <= n; ++k) seq_begin[k] = pl.seq_begin[k];
  return n;
}

size_t policy_loss_workspace(const fastrl_loss_args& a) {
  SlabPlan pl = plan_slabs(a.seq_off_host, a.S, slab_cap(a));
  Carver c(nullptr);
  LossWs w;
  return carve_loss(c, w, a, pl);
}

template <typename T>
static int policy_loss_impl(const fastrl_loss_args& a, hipStream_t stream) {
  SlabPlan pl = plan_slabs(a.seq_off_host, a.S, slab_cap(a));
  Carver c(a.ws);
  LossWs w;
  carve_loss(c, w, a, pl);
  const int64_t Vpad = rup(a.V, kBM);
  const int64_t tcp = rup(std::max<int64_t>(pl.tc_max, 1), kBN);
  const int32_t nmb = int32_t(Vpad / kBM);
  const bool dh = a.dhidden != nullptr, dw = a.dW != nullptr;
  const int32_t d = a.d, V = a.V;

  // no token at all (S == 0, or only empty sequences): no slab clears the count or writes dW
  if (a.T == 0) {
    hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(64), 0, stream, w.redo_count, int64_t(1), 0);
    FR_LAUNCHED();
  }
  if (dw && !a.dW_accumulate && a.T == 0) {
    hipLaunchKernelGGL(fill_i32_kernel, dim3(1024), dim3(256), 0, stream,
                       reinterpret_cast<int32_t*>(a.dW), int64_t(V) * d, 0);
    FR_LAUNCHED();
  }
  const bool direct = direct_dh(a);
  if (dh && !direct && a.S > 0) {
    dim3 g(nb1d(d, 64), unsigned(Vpad / 64));
    hipLaunchKernelGGL(transpose_scale_kernel, g, dim3(256), 0, stream,
                       static_cast<const uint16_t*>(a.W), (const int32_t*)nullptr, int64_t(0), V,
                       int32_t(Vpad), d, (const float*)nullptr, static_cast<uint16_t*>(w.WT), Vpad);
    FR_LAUNCHED();
  }
  const size_t nslab = pl.seq_begin.size() - 1;
  LossParams lp{};
  lp.logp = w.logp; lp.lse = w.lse; lp.ent = w.ent;
  lp.old_logp = a.old_logp; lp.ref_logp = a.ref_logp; lp.row_index = a.row_index;
  lp.seq_off = a.seq_off; lp.adv = a.adv; lp.seq_index = a.seq_index;
  lp.S = a.S; lp.T = a.T; lp.algo = a.algo; lp.norm = a.norm;
  lp.eps_low = a.eps_low; lp.eps_high = a.eps_high; lp.beta = a.beta;
  lp.shift = dh || dw ? w.shift : nullptr; lp.cslab = w.cslab;
  lp.seq_loss = w.seq_loss; lp.seq_clip = w.seq_clip; lp.status = a.status;
  lp.nadv = a.seq_index ? INT32_MAX : a.S;
  lp.E1 = dh || dw ? w.E1 : nullptr; lp.ldE1 = Vpad; lp.e_bf16 = sizeof(T) == 2;
  lp.yslab = w.yslab; lp.psum = w.psum; lp.psz = w.psz; lp.zlab = w.zlab;
  lp.ldp = tcp; lp.nmb = nmb;
  lp.redo_count = w.redo_count; lp.loss = a.loss; lp.stats = a.stats;
  bool dw_written = false;  // a slab's dW GEMM has overwritten dW
  for (size_t si = 0; si < nslab; ++si) {
    const int32_t s0 = pl.seq_begin[si], s1 = pl.seq_begin[si + 1];
    const int64_t t0 = a.seq_off_host[s0];
    const int32_t Tc = int32_t(a.seq_off_host[s1] - t0);
    lp.seq_begin = s0;
    lp.row_base = t0;
    if (Tc == 0) {  // only empty sequences (T == 0): their loss terms and clip counts are 0
      FR_TRY(launch_loss(lp, s1 - s0, 0, 0, stream));
      continue;
    }
    const int32_t nnb = int32_t(rup(Tc, kBN) / kBN);
    hipLaunchKernelGGL(slab_prep_kernel, dim3(nb1d(Tc, 256)), dim3(256), 0, stream,
                       a.token_ids, a.row_index, t0, Tc, V, w.yslab, w.shift, a.status,
                       w.redo_blk, nnb + 1, si == 0 ? w.redo_count : (int32_t*)nullptr);
    FR_LAUNCHED();
    GemmParams p{};
    p.A = a.W; p.lda = d; p.M = V;
    p.B = a.hidden; p.ldb = d; p.N = Tc; p.b_rows = a.row_index; p.b_row_base = t0;
    p.K = d;
    p.pmax = w.pmax; p.psum = w.psum; p.psz = w.psz; p.ldp = tcp; p.zlab = w.zlab;
    p.yslab = w.yslab; p.shift = w.shift; p.E1 = w.E1; p.ldE1 = Vpad;
    p.Vreal = V; p.store_e = (dh || dw) ? 1 : 0;
    p.redo_blk = w.redo_blk;
    p.redo_any = w.redo_blk + nnb;
    const double f_fwd = 2.0 * double(V) * Tc * d;
    FR_TRY((launch_gemm<T, MODE_FWD>(p, FASTRL_K_LOGITS_FWD, f_fwd, stream)));
    const bool store = dh || dw;
    FR_TRY(launch_merge(w.pmax, w.psum, w.psz, tcp, nmb, w.zlab, w.yslab, Tc, store, w.lse + t0,
                        w.logp + t0, w.ent ? w.ent + t0 : nullptr, store ? w.shift : nullptr,
                        w.redo_blk, w.redo_count, w.redo_blk + nnb, stream));
    // token blocks holding a row that needs a shift: evaluate again (returns at once on the device
    // when no row was marked); loss_kernel merges those rows
    if (store) FR_TRY(launch_redo<T>(p, stream));
    lp.redo_any = w.redo_blk + nnb;
    int64_t longest = 0;
    for (int32_t i = s0; i < s1; ++i)
      longest = std::max(longest, a.seq_off_host[i + 1] - a.seq_off_host[i]);
    FR_TRY(launch_loss(lp, s1 - s0, Tc, longest, stream));
    GemmParams q{};  // dhidden: C = E W^T (rows = tokens, cols = d, K = padded vocabulary)
    if (dh) {
      q.A = w.E1; q.lda = Vpad; q.M = Tc;
      q.B = w.WT; q.ldb = Vpad; q.N = d;
      q.K = int32_t(Vpad);
      q.dH = a.dhidden_dtype == FASTRL_BF16
                 ? (void*)(static_cast<uint16_t*>(a.dhidden) + t0 * d)
                 : (void*)(static_cast<float*>(a.dhidden) + t0 * d);
      q.dH_bf16 = a.dhidden_dtype == FASTRL_BF16;
      q.cslab = w.cslab; q.d = d;
      if (direct) {
        q.B = a.W; q.ldb = d; q.K = int32_t(rup(V, sizeof(T) == 2 ? 64 : BK_F32)); q.Vreal = V;
        q.ksplit = dh_ksplit(Tc, d, V, a.dtype, dw);
        q.part = static_cast<float*>(w.WT);
      }
    }
    // bf16 with both gradients: the two GEMMs run as one launch (after dW's inputs are ready)
    const bool wide = sizeof(T) == 2 && (Vpad >= kMaxLd || (dw && tcp >= kMaxLd));
    const bool fused = dh && dw && sizeof(T) == 2 && !wide;
    if (dh && wide && direct)
      FR_TRY(launch_wide<MODE_DHT>(q, FASTRL_K_DHIDDEN, 2.0 * double(Tc) * d * V, stream));
    else if (dh && !dw && direct && sizeof(T) == 2)
      FR_TRY(launch_bwd_direct(q, GemmParams{}, false, 2.0 * double(Tc) * d * V, stream));
    else if (dh && !fused)
      FR_TRY((launch_gemm<T, MODE_DH>(q, FASTRL_K_DHIDDEN, 2.0 * double(Tc) * d * V, stream)));
    if (dw) {
      GemmParams r{};
      r.dW = a.dW; r.dW_acc = (dw_written || a.dW_accumulate) ? 1 : 0;
      r.d = d;
      if constexpr (sizeof(T) == 2) {  // dW^T = Bd E: A = Bd, B = E1 read K-major
        // (the logits tiles zero the exp-logit rows up to a multiple of 64 tokens)
        const int64_t Tr = rup(Tc, 64);
        dim3 g(nb1d(d, 64), unsigned(Tr / 64));
        hipLaunchKernelGGL(transpose_scale_kernel, g, dim3(256), 0, stream,
                           static_cast<const uint16_t*>(a.hidden), a.row_index, t0, Tc, int32_t(Tr),
                           d, w.cslab, static_cast<uint16_t*>(w.Bd), tcp);
        FR_LAUNCHED();
        r.K = int32_t(Tr);
        r.A = w.Bd; r.lda = tcp; r.M = d;
        r.B = w.E1; r.ldb = Vpad; r.N = V;
        if (fused && direct)
          FR_TRY(launch_bwd_direct(q, r, true, 4.0 * double(V) * d * Tc, stream));
        else if (fused)
          FR_TRY(launch_bwd(q, r, 4.0 * double(V) * d * Tc, stream));
        else
          FR_TRY((launch_gemm<T, MODE_DWT>(r, FASTRL_K_DW, 2.0 * double(V) * d * Tc, stream)));
      } else {  // dW = E^T Bd: A = E1 and B = Bd (here c_t H[t] as rows) both read K-major
        r.K = int32_t(rup(Tc, BK_F32));
        const int64_t n4 = int64_t(r.K) * (d / 4);
        hipLaunchKernelGGL(scale_rows_f32_kernel,
                           dim3(unsigned(std::min<int64_t>((n4 + 255) / 256, 4 * kMaxBlocks))),
                           dim3(256), 0, stream,
                           static_cast<const float*>(a.hidden), a.row_index, t0, Tc, r.K, d,
                           w.cslab, static_cast<float*>(w.Bd));
        FR_LAUNCHED();
        r.A = w.E1; r.lda = Vpad; r.M = V;
        r.B = w.Bd; r.ldb = d; r.N = d;
        FR_TRY((launch_gemm<T, MODE_DW>(r, FASTRL_K_DW, 2.0 * double(V) * d * Tc, stream)));
      }
      dw_written = true;
    }
  }
  hipLaunchKernelGGL(loss_final_kernel, dim3(1), dim3(kSumThreads), 0, stream, lp);
  FR_LAUNCHED();
  if (a.entropy_sum) {
    hipLaunchKernelGGL(sum_f32_kernel, dim3(1), dim3(kSumThreads), 0, stream, w.ent, a.T,
                       a.entropy_sum);
    FR_LAUNCHED();
  }
  return FASTRL_OK;
}

int run_policy_loss(const fastrl_loss_args& a, hipStream_t stream) {
  if (a.dtype == FASTRL_BF16) return policy_loss_impl<uint16_t>(a, stream);
  return policy_loss_impl<float>(a, stream);
}

}  // namespace fastrl
