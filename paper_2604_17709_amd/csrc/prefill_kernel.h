// Compute-bound ("prefill", T > 128 tokens) kernel for PACKED bf16 factor pairs.
//
// Both stages of y = (x U) V (Sec. 4.1) are the same "NT" GEMM  out[T x F] = act[T x K] . W^T
// with the weights W[F x K] in packed MFMA-fragment order:
//   stage 1  act = x,  W = [U_a | U_b | U_c]^T (concatenated feature axis), out = t (bf16, one
//            nearest-even rounding, row-major so that it is stage 2's activation operand);
//   stage 2  act = t,  W = V^T of one pair, out = y.  The GLU call computes both products of a
//            tile in one workgroup, one after the other on the same accumulators: the gate product,
//            then silu of it rounded to the storage type into 128 registers that the main loop
//            leaves free, then the up product, whose epilogue multiplies the two: the full-width
//            gate and up results never leave the registers (a side-by-side accumulation, half the
//            tile per product, would need 1.5 x the LDS traffic per flop).
// t makes one round trip through HBM / Infinity Cache (<= 75 MB, a few percent of the MFMA
// time); a 256-row t tile does not fit the 160 KB LDS at these ranks.
//
// Tiling: 256 threads = 4 wavefronts (2 x 2), one per SIMD, workgroup tile 256 tokens x
// (32 * MF) features; each wavefront owns 128 tokens x (16 * MF) features as MF x 8 accumulator
// blocks of the 16x16x32 MFMA (features = MFMA rows, tokens = MFMA columns).  MF = 8 uses all 256
// accumulation registers.
// Both operands go from global memory straight into LDS (buffer loads with the LDS modifier,
// 16 bytes per lane, 1 KiB contiguous in LDS per wavefront instruction, no staging registers):
// weight fragments are already contiguous 1 KiB pieces; activations come as 128-byte token rows,
// the two k-blocks of a pair of stages at once, whose eight 16-byte slots are XOR-swizzled with
// (row / 2) % 8, applied on the global side of the load (lane -> slot is fixed, lane -> k-chunk is
// permuted), which keeps the operand reads free of bank conflicts without padding (SQ_LDS_BANK_CONFLICT is 0 in the
// k-split launches, which use LDS for nothing else; the epilogue's transpose costs the others 1-8 % of their LDS cycles).
// What bounds the loop beside the products is the number of requests to L2.  One k-block per row
// and load (64 bytes, half a cache line) made every row two requests: 384 per 256 x 256 tile and
// stage; whole lines make it 256 (70B GLU launch: TCP_TCC_READ_REQ_sum 73.4 M over 1792 tiles of 160
// stages).  7B block, 512 tokens 295 -> 271 us (its GLU
// launch 70 -> 61 us), 8192 tokens 1749 -> 1627 us; 70B at 4096 tokens 2426 -> 2321 us; 13B at 8256
// 2820 -> 2740 us; cached keys and values of 8192 tokens 243 -> 230 us.  (Rows whose pitch or first
// column is no multiple of 128 bytes keep part of the second requests.)
// Pipeline: one stage = one 32-wide k-block; the weights of stage s + 3 and half of the activations
// of the pair that starts three or four stages later are requested while stage s is multiplied
// (four weight buffers of 16 KiB, three activation buffers of 32 KiB: all 160 KiB of LDS); one
// barrier per stage, placed in the middle of the stage's products so that the feature fragments of
// stage s + 1 can be read from LDS during the second half of stage s.
#pragma once
#include <type_traits>
#include "common.h"

namespace deinfer {

#if defined(__HIP_DEVICE_COMPILE__)
#define DEINFER_GLOBAL __attribute__((address_space(1)))
#define DEINFER_LOCAL __attribute__((address_space(3)))
#else
#define DEINFER_GLOBAL
#define DEINFER_LOCAL
#endif

constexpr int PF_THREADS = 256;
constexpr int PF_BT = 256;                 // tokens per workgroup tile
constexpr int PF_BK = 32;                  // k per pipeline stage (one k-block)
constexpr int PF_STAGES = 4;               // LDS stage buffers of the 256-token tile
constexpr int PF_STAGES_TB2 = 6;           // ... of the 128 x 256 tile (half the products per stage: a deeper queue for the same cover)
constexpr int PF_STAGES_MF4 = 6;           // ... of the 128 x 128 tile (blocks of 200 to 1024 tokens, where both small tiles run,
                                           // are 7-14 % slower with four stages for both, 1-4 % slower with eight for this one)
constexpr int pf_stages(int tb, int mf = 8) { return tb == 4 ? PF_STAGES : mf == 8 ? PF_STAGES_TB2 : PF_STAGES_MF4; }

// Launches with at most this many token blocks give every XCD (workgroup index mod 8) a contiguous run of tiles:
// the token blocks of a feature block then share one L2, which fetches the weights once; dealt out in turn,
// every token block's XCD fetches them for itself (4 x the weights at 4 token blocks).  With 16 or more token
// blocks a run would hold as many activation panels as the other order holds weight panels.
constexpr int PF_RUN_TBLOCKS = 8;
constexpr int PF_XPITCH = PF_BK * 4;       // bytes per token row of the activation tile in LDS: the k-blocks of two stages
constexpr int pf_xpairs(int tb, int mf = 8) { return pf_stages(tb, mf) / 2 + 1; }     // activation buffers (two stages each)

struct PfSeg {             // a run of 16-feature tiles that belongs to one factor
  const uint4 *frags;      // its packed fragments [tiles][KB][64]
  int tile0;               // first tile of the segment on the concatenated feature axis
  int width2;              // optional second copy of the segment's first width2 columns (rank-space output) ...
  uint16_t *out2;          // ... or null; 16-byte aligned rows (plain products only: no GLU, POST, ROPE, SPLIT)
  long long ldo2;
};

struct PfProblem {         // one product  act[T x K] . W^T
  const uint16_t *act;     // row-major bf16
  long long lda;
  int K;                   // valid k (columns of act)
  int KB;                  // 32-wide k-blocks of the packed weights (zero padded)
  int n_seg;
  PfSeg seg[3];
  int n_ftiles;            // 16-feature tiles on the (concatenated) feature axis
  uint16_t *out;           // output [T x width] bf16 row-major: feature tile g lands at columns 16 g ..
  long long ldo;
  int width;               // valid output columns
  const uint16_t *bias;    // POST kernels only: out = act(product + bias[column]); may be null
  int post_act;            // see act_f32
  const float *rope;       // ROPE kernels only: [T][128] cos | sin of the rotary angles (heads of 128 features)
};

struct PfParams {
  int T;
  int n_tblocks;           // ceil(T / 256)
  // Up to three independent products in one launch (the upward projections of a q/k/v call: a
  // narrow one alone would leave most of the device idle); product i owns the feature blocks
  // [fb0[i], fb0[i + 1]) of the grid.
  int n_prob;
  int fb0[3];
  PfProblem prob[3];
  // SPLIT kernels only (few tiles, long k: the k range is cut into parts, one workgroup per part)
  int n_fblocks;           // feature blocks of 256; grid = n_tblocks * n_fblocks * n_parts
  int kb_per_part;         // k-blocks per part
  float *part;             // [n_parts][n_tblocks * 256][n_fblocks * 256] fp32 partial products
  long long part_stride;   // elements between parts
  // prefill_mixed_kernel only
  int n_big;               // workgroups with 256 x 256 tiles (they come first)
  int n_tblocks2;          // ceil(T / 128): token blocks of the 128 x 256 tiles
  int fb_shift2;           // first feature block (of 256 features) of the 128 x 256 tiles
};

template <int MF, int TB = 4>
struct PfShared {
  uint4 w[pf_stages(TB, MF)][2 * MF][64];                   // [stage][feature tile][lane]
  unsigned char x[pf_xpairs(TB, MF)][64 * TB * PF_XPITCH];  // [pair of stages][token row * 128 bytes], slots swizzled
};

// GLU = true: two products per tile, P.prob[0] (gate) and P.prob[1] (up, same feature tiles and output):
// out = silu(gate product) * up product.
// POST = PF_POST_BIAS_ACT: bias and activation of the non-GLU MLP sub-layer on the fp32 accumulators;
// PF_POST_TAIL: the activation rows' valid columns K may be no multiple of 8 (the caller's rank-space rows
// of an upward projection alone): what the last chunk holds beyond column K - 1 is set to zero in LDS.
// SPLIT = true: this workgroup multiplies only its part of the k range and stores the fp32
// accumulators to a partial buffer (the sum and the epilogue are a second, small kernel's).
// DT = storage type of weights, activations and outputs (DT_BF16 or DT_F16).
// ROPE = true: rotary embedding of the output (heads of 128 features = one wavefront's features:
// feature i of a head pairs with feature i + 64 of the same token, both in this wavefront's LDS
// tile), on the rounded products, cos / sin from a table; the result is rounded once more.
// TB = 32-token blocks per wavefront: 4 (workgroup tile of 256 tokens) or 2 (128 tokens: twice the
// workgroups, for launches whose 256-token tiles are fewer than the compute units; the same stage schedule with
// half the groups and a deeper queue).
// The body of a workgroup: bid = its index among the workgroups of this tile shape, n_tblocks = token
// blocks of this tile shape, fb_shift = first feature block of this tile shape (0 unless the launch
// mixes two shapes, see prefill_mixed_kernel).
constexpr int PF_POST_NONE = 0, PF_POST_BIAS_ACT = 1, PF_POST_TAIL = 2;

template <int DT, int MF, bool GLU, int POSTK, bool SPLIT, bool ROPE, int TB>
__device__ __forceinline__ void prefill_body(const PfParams &P, const int bid, const int n_tiles, const int n_tblocks, const int fb_shift) {
  constexpr bool POST = POSTK == PF_POST_BIAS_ACT, TAIL = POSTK == PF_POST_TAIL;
  static_assert(!(ROPE && (GLU || POST || SPLIT)), "the rotary epilogue goes with a plain product");
  static_assert(!(TAIL && SPLIT), "only a second stage reads caller rows");
  static_assert(TB == 4 || (TB == 2 && !SPLIT), "token blocks per wavefront");
#if defined(__HIP_DEVICE_COMPILE__)      // the body uses device-only builtins; the host pass only needs the stub
  constexpr int WTOK = 32 * TB;                    // tokens per wavefront
  constexpr int BT = 2 * WTOK;                     // tokens per workgroup tile
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  PfShared<MF, TB> &S = *reinterpret_cast<PfShared<MF, TB> *>(smem_raw);
  constexpr int NST = pf_stages(TB, MF);           // LDS stage buffers; loads run NST - 1 stages ahead
  constexpr int BF_TILES = 2 * MF;                 // 16-feature tiles per workgroup
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wf = wave & 1, wt = wave >> 1;         // wavefront position: features x tokens

  // Tiles in order share a feature block and differ in the token block.  Workgroups go to the eight XCDs
  // in turn, so with a multiple of 8 token blocks an XCD keeps a few token blocks and runs through the
  // features.  With few token blocks (run_tile_of) every XCD takes a contiguous run of tiles instead.
  const int tile = n_tblocks <= PF_RUN_TBLOCKS ? run_tile_of(bid, n_tiles) : bid;
  const int tb = tile % n_tblocks;
  const int fb_all = tile / n_tblocks + fb_shift;
  int fb = SPLIT ? fb_all % P.n_fblocks : fb_all;
  int pi = 0;                                                   // which product (uniform)
  if (!SPLIT && P.n_prob > 1 && fb >= P.fb0[1]) pi = 1;
  if (!SPLIT && P.n_prob > 2 && fb >= P.fb0[2]) pi = 2;
  fb -= P.fb0[pi];
  const int kpart = SPLIT ? fb_all / P.n_fblocks : 0;
  const int kb0 = SPLIT ? kpart * P.kb_per_part : 0;          // first k-block of this workgroup
  const int tok0 = tb * BT;

  constexpr int TJ = 2 * TB;                       // 16-token blocks per wavefront (MF 16-feature blocks)
  static_assert((MF == 8 || (MF == 4 && TB == 2 && !ROPE)) && (TB == 4 || TB == 2), "wavefront tiles the stage schedule is written for");
  f32x4_t acc[MF][TJ];                             // [feature block][token block]
#pragma unroll
  for (int i = 0; i < MF; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // GLU: silu(gate product), rounded once to the storage type, kept in registers (as pairs) while the
  // up product is accumulated: element [i][j] holds the four values of accumulator block (i, j)
  uint2 gpk[GLU ? MF : 1][GLU ? TJ : 1];
  // One product of this workgroup's tile: acc += act . W^T over the whole k range of Q.  between() runs
  // once the first pipeline stages have been requested and before they are waited for.
  auto product = [&](const PfProblem &Q, auto &&between) {
    // ---- load assignment (every instruction moves 1 KiB: lane l -> LDS base + 16 l).
    // Buffer addressing: a scalar resource descriptor, a scalar byte offset for the k position
    // and one 32-bit per-lane offset, which leaves the registers to the accumulators; reads
    // beyond a descriptor's size (token rows >= T, feature tiles past the last one) return
    // zeros instead of faulting.  (Host guarantees every tensor here is below 2^31 bytes.)
    constexpr int WT = BF_TILES / 4;       // feature tiles fetched per wavefront and stage
    constexpr int LPS = WT + TB;           // load instructions per wavefront and stage
    const int uwave = __builtin_amdgcn_readfirstlane(wave);
    __amdgpu_buffer_rsrc_t wres[WT];
    unsigned wtile_off[WT];
#pragma unroll
    for (int i = 0; i < WT; ++i) {
      const int gt = fb * BF_TILES + uwave * WT + i;
      int sgi = 0;
      if (Q.n_seg > 1 && gt >= Q.seg[1].tile0) sgi = 1;
      if (Q.n_seg > 2 && gt >= Q.seg[2].tile0) sgi = 2;
      const int seg_end = sgi + 1 < Q.n_seg ? Q.seg[sgi + 1].tile0 : Q.n_ftiles;
      // a feature tile past the last one gets an empty descriptor: every read of it returns zeros
      const bool live = gt < Q.n_ftiles;
      wres[i] = __builtin_amdgcn_make_buffer_rsrc((void *)Q.seg[sgi].frags, 0,
                                                  live ? (int)((unsigned)(seg_end - Q.seg[sgi].tile0) * (unsigned)Q.KB * 1024u) : 0, 0x00020000);
      wtile_off[i] = live ? (unsigned)(gt - Q.seg[sgi].tile0) * (unsigned)Q.KB * 1024u : 0u;
    }
    const unsigned wlane = lane * 16;
    // activations: both k-blocks of a pair of stages at once, whole 128-byte lines.  Instruction i (0 .. 2 TB - 1)
    // of wavefront w covers tile rows 8 (4 i + w) .. + 7; lane l holds slot l % 8 of row l / 8 and fetches k-chunk
    // slot ^ (row / 2) % 8 = (l & 7) ^ (4 (w & 1) + l / 16)
    const __amdgpu_buffer_rsrc_t xres =
        __builtin_amdgcn_make_buffer_rsrc((void *)Q.act, 0, (int)((unsigned)P.T * (unsigned)(Q.lda * 2)), 0x00020000);
    const int chunk = (lane & 7) ^ (((wave & 1) << 2) | (lane >> 4));
    const unsigned xrow = (unsigned)(tok0 + 8 * wave + (lane >> 3)) * (unsigned)(Q.lda * 2);
    const unsigned xstep = 32u * (unsigned)(Q.lda * 2);
    const int n_stages = SPLIT ? (Q.KB - kb0 < P.kb_per_part ? Q.KB - kb0 : P.kb_per_part) : Q.KB;

    constexpr int D = NST - 1;             // weight loads run D stages ahead of the products
    constexpr int XM = (D + 1) / 2;        // activation loads run XM pairs of stages ahead
    constexpr int NXP = pf_xpairs(TB, MF);
    static_assert(NXP == XM + 1, "the buffer of the pair before is free");
    constexpr unsigned DEAD = 0x80000000u; // lane offset of an activation load that is not needed: beyond every descriptor, reads zeros
    // One load instruction (index 0 .. LPS - 1) of slot sl, the loads that go out beside the products of stage sl:
    // the weight tiles of stage sl + D, then the first (sl even) or second half of the activation rows of pair
    // sl / 2 + XM.  Every slot issues all of its loads, those past the last stage as dead ones that read zeros: the
    // load counter is the same in every stage.
    // Activation chunks beyond K re-read a chunk of valid columns (the last one; PF_POST_TAIL: the first one),
    // which meets zero weights.
    const unsigned xchunk = (unsigned)(chunk * 16);
    const unsigned xkend = (unsigned)(((Q.K + 7) >> 3) * 16);    // bytes of a row up to the end of the chunk that holds column K - 1
    const unsigned xklim = (unsigned)(Q.K * 2 - 16);             // (K a multiple of 8: the last chunk)
    // Valid columns K that are no multiple of 8 (the caller's rank-space rows of an upward projection alone):
    // the stage whose tile holds the chunk with column K - 1; once it has landed, the elements of that chunk
    // beyond K - 1 are set to zero (lds_zero_chunk_tail in common.h).  -1: nothing to do (every other call).
    const int krem = Q.K & 7;
    const int st_fix = (TAIL && krem != 0) ? (Q.K >> 5) - kb0 : -1;
    auto fix_tail = [&] {
      if constexpr (TAIL) {
        int row = threadIdx.x;
        asm volatile("" : "+v"(row));
        if (row < 64 * TB)
          lds_zero_chunk_tail(&S.x[(st_fix >> 1) % NXP][row * PF_XPITCH + (((4 * (st_fix & 1) + ((Q.K >> 3) & 3)) ^ ((row >> 1) & 7)) * 16)], krem);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
    };
    auto fetch_part = [&](int sl, int idx, auto sure) {          // sure: the stages it belongs to exist
      constexpr bool SURE = decltype(sure)::value;
      if (idx < WT) {
        const int st = sl + D;
        const BufOffsets off = weight_load(SURE || st < n_stages, wlane, wtile_off[idx] + (unsigned)(st + kb0) * 1024u);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(wres[idx], (DEINFER_LOCAL void *)&S.w[st % NST][uwave * WT + idx][0], 16, off.lane, off.scalar, 0, 0);
      } else {
        const int pair = (sl >> 1) + XM, i = (sl & 1) * TB + idx - WT;
        const unsigned dead = SURE || 2 * pair < n_stages ? 0u : DEAD;
        unsigned kb = (unsigned)(2 * pair + kb0) * (PF_BK * 2) + xchunk;
        kb = TAIL ? (kb < xkend ? kb : 0u) : (kb < xklim ? kb : xklim);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (DEINFER_LOCAL void *)&S.x[pair % NXP][8 * (4 * i + uwave) * PF_XPITCH], 16,
                                                 (xrow + (unsigned)i * xstep + kb) | dead, 0, 0, 0);
      }
    };
    // Operand reads for the 16x16x32 product: lane l works on row (feature or token) l % 16 and on the 8
    // consecutive k of group l / 16.  A packed 16-feature fragment is in that order already.
    // A row's two k-blocks: slots 0 .. 3 and 4 .. 7 before the swizzle, i.e. 64 bytes apart by exclusive or.  The
    // swizzle keeps the 16 lanes that the LDS serves at once (0-3, 12-15, 20-27 and so on: two k-groups) on 16
    // different groups of four banks.
    const int b_off = (wt * WTOK + (lane & 15)) * PF_XPITCH + (((lane >> 4) ^ ((lane >> 1) & 7)) * 16);
    auto read_a = [&](int buf, int i) -> u32x4_t { return *reinterpret_cast<const u32x4_t *>(&S.w[buf][wf * MF + i][lane]); };
    auto read_b = [&](int xbuf, int odd, int j) -> u32x4_t {
      return *reinterpret_cast<const u32x4_t *>(&S.x[xbuf][(b_off ^ (64 * odd)) + 16 * j * PF_XPITCH]);
    };
    constexpr int H1 = LPS / 2;            // loads 0 .. H1 - 1 of slot s go out in the second half of stage s,
                                           // loads H1 .. LPS - 1 in the first half of stage s + 1
    const std::true_type yes;
    const std::false_type no;
    static_assert((D - 2) * LPS + H1 < 64, "the load counter has 6 bits");
    // the first half of pair 0, slots -D .. -2 whole and the first half of slot -1, then wait for stage 0
#pragma unroll
    for (int i = WT; i < LPS; ++i) fetch_part(-D - 1, i, yes);
#pragma unroll
    for (int sl = -D; sl < -1; ++sl) {
#pragma unroll
      for (int i = 0; i < LPS; ++i) fetch_part(sl, i, no);
    }
#pragma unroll
    for (int i = 0; i < H1; ++i) fetch_part(-1, i, no);
    between();
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 2) * LPS + H1) : "memory");    // slot -D has arrived
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();          // stage 0 has landed everywhere
    asm volatile("" ::: "memory");
    if constexpr (TAIL) {
      if (st_fix == 0) fix_tail();
    }
    // A stage is TJ groups of MF products that share one token operand (a group: 16 cycles per product).
    // Token operands are read two groups ahead of their use into a ring of four, the feature operands of
    // the next stage during the second half of this one.
    u32x4_t a0[MF], a1[MF], b[4];
#pragma unroll
    for (int i = 0; i < MF; ++i) a0[i] = read_a(0, i);
    b[0] = read_b(0, 0, 0);
    b[1] = read_b(0, 0, 1);
    // One stage: feature operands in `a`, those of the next stage into `an`; odd = st % 2.  STEADY: every stage
    // that the slot's loads belong to exists.  At most two memory instructions follow a product: their issue
    // hides behind the products' cycles in the matrix pipeline.
    auto stage = [&](int st, u32x4_t (&a)[MF], u32x4_t (&an)[MF], auto odd_t, auto steady) {
      constexpr bool STEADY = decltype(steady)::value;
      constexpr int ODD = decltype(odd_t)::value;
      const int nbuf = (st + 1) % NST;
      const int xbuf = (st >> 1) % NXP, nxbuf = ((st + 1) >> 1) % NXP;
      constexpr int HG = TJ / 2, HN = HG * MF;             // groups / products of half a stage
      constexpr int AN = MF / HG;                          // next-stage feature operands read per group of the second half
      auto half = [&](auto second) {
        constexpr bool SECOND = decltype(second)::value;
        constexpr int NL = SECOND ? H1 : LPS - H1;         // load requests of this half
#pragma unroll
        for (int gg = 0; gg < HG; ++gg) {
          const int g = gg + (SECOND ? HG : 0);
#pragma unroll
          for (int i = 0; i < MF; ++i) {
            const int n = gg * MF + i;
            mfma16_acc<DT>(a[i], b[g & 3], acc[i][g]);
#pragma unroll
            for (int l = 0; l < NL; ++l)
              if (l * HN / NL == n) {
                if (SECOND) fetch_part(st, l, steady);
                else fetch_part(st - 1, H1 + l, steady);
              }
            if (i == 1) b[(g + 2) & 3] = g + 2 < TJ ? read_b(xbuf, ODD, g + 2) : read_b(nxbuf, 1 - ODD, g + 2 - TJ);
            if (SECOND) {
#pragma unroll
              for (int t = 0; t < AN; ++t)
                if (i == 2 + t * (MF - 2) / AN) an[gg * AN + t] = read_a(nbuf, gg * AN + t);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      };
      half(std::false_type{});
      // stage st + 1 has landed (this wavefront's part) once at most the loads of the slots st - D + 2 .. st - 1 are
      // outstanding (its weights are in slot st + 1 - D, its activations in slots up to that one); after the
      // barrier it has landed everywhere and nobody reads the weights of stage st - 1 or the activations of the
      // pair before this one any more, whose buffers slot st fills.  A bare barrier: the wait is the only ordering
      // needed (loads into LDS are complete when the counter says so); the fence of __syncthreads() would drain
      // every outstanding load instead.
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 2) * LPS) : "memory");
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      // (the chunk that holds column K - 1 is in the last stage: only stages without a whole pipeline behind
      // them can precede it, so the steady-state loop carries no branch for this)
      if constexpr (TAIL && !STEADY) {
        if (st + 1 == st_fix) fix_tail();                  // (uniform)
      }
      // (after the last stage the reads ahead hit a stage buffer nobody writes any more; the values are unused)
      half(std::true_type{});
    };
    {
      const std::integral_constant<int, 0> even;
      const std::integral_constant<int, 1> odd;
      int st = 0;
      // (the loads of slot st + 1: weights of stage st + 1 + D, activations of stages up to st + 2 XM + 1 = st + D + 2;
      // the last of these may not exist: its columns are clamped to the row's valid ones and are not multiplied)
      for (; st + 1 + D < n_stages; st += 2) {
        stage(st, a0, a1, even, yes);
        stage(st + 1, a1, a0, odd, yes);
      }
      for (; st < n_stages; st += 2) {
        stage(st, a0, a1, even, no);
        if (st + 1 >= n_stages) break;
        stage(st + 1, a1, a0, odd, no);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the dead loads write zeros: before anything else uses the buffers
    mfma_settle(acc);
  };
  if constexpr (GLU) {
    // Both products of the tile in this workgroup (Sec. 4.1: gate and up share x and the output
    // columns): the gate product first; its silu goes into registers while the up product's first
    // stages are on their way; the full-width gate and up results never reach memory.
    product(P.prob[0], [] {});
    __syncthreads();       // every wavefront has read its last gate-product operands: the stage buffers are free
    product(P.prob[1], [&] {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          // (the sums are taken out of the accumulator registers here, by hand: the compiler would
          // move all 256 of them to ordinary registers at the end of the gate product's loop, where
          // they would have to live through the requests above)
          float z[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(z[e]) : "a"(acc[i][j][e]));
            acc[i][j][e] = 0.f;
          }
          gpk[i][j].x = pack2<DT>(silu_f32(z[0]), silu_f32(z[1]));
          gpk[i][j].y = pack2<DT>(silu_f32(z[2]), silu_f32(z[3]));
          // (the packed values are made opaque here: otherwise the compiler defers silu to the
          // epilogue and keeps all 256 raw gate sums alive through the second product's loop)
          asm volatile("" : "+v"(gpk[i][j].x), "+v"(gpk[i][j].y));
        }
    });
  } else {
    product(P.prob[pi], [] {});
  }
  const PfProblem &Q = P.prob[pi];         // (GLU: the gate problem; output buffer and width are the same for both)
  // (lane-derived values are taken afresh so that none has to live through the main loop)
  int tid_e = threadIdx.x;
  asm volatile("" : "+v"(tid_e));
  const int lane_e = tid_e & 63, wave_e = tid_e >> 6, wf_e = wave_e & 1, wt_e = wave_e >> 1;
  if constexpr (SPLIT) {
    // element e of block (i, j) is feature 16 i + 4 (lane / 16) + e, token 16 j + lane % 16: four
    // consecutive features = one 16-byte store; the buffer has whole tiles, no bounds to check
    const long long F = (long long)P.n_fblocks * (32 * MF);
    float *dst = P.part + (long long)kpart * P.part_stride + (long long)(tok0 + wt_e * WTOK + (lane_e & 15)) * F +
                 (fb * BF_TILES + wf_e * MF) * 16 + 4 * (lane_e >> 4);
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) *reinterpret_cast<f32x4_t *>(dst + (long long)(16 * j) * F + 16 * i) = acc[i][j];
    return;
  }
  // accumulators -> bf16 pairs first (registers only): it overlaps the wait for the slowest wavefront.
  // (GLU and POST: not ahead of the barrier.  128 registers of pairs do not fit beside the 128 of the gate values,
  // nor, without a spill, beside the activation's temporaries: every pair is formed right before it is written to
  // LDS instead)
  constexpr bool LATE = GLU || POST;
  uint2 pk[LATE ? 1 : MF][LATE ? 1 : TJ];
  if constexpr (!LATE) {
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        pk[LATE ? 0 : i][LATE ? 0 : j].x = pack2<DT>(acc[i][j][0], acc[i][j][1]);
        pk[LATE ? 0 : i][LATE ? 0 : j].y = pack2<DT>(acc[i][j][2], acc[i][j][3]);
      }
  }
  // POST: the bias of this lane's features, four per feature block, on the way while the barrier is waited for:
  // element e of block (i, j) is feature 16 i + 4 (lane / 16) + e of this wavefront's 16 MF features
  uint2 bias[POST ? MF : 1];
  if constexpr (POST) {
#pragma unroll
    for (int i = 0; i < MF; ++i) {
      const int f0 = (fb * BF_TILES + wf_e * MF) * 16 + 16 * i + 4 * (lane_e >> 4);
      uint16_t b[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = Q.bias != nullptr && f0 + e < Q.width ? Q.bias[f0 + e] : (uint16_t)0;
      bias[POST ? i : 0] = make_uint2((unsigned)b[0] | ((unsigned)b[1] << 16), (unsigned)b[2] | ((unsigned)b[3] << 16));
    }
  }

  // ---- epilogue: through LDS (free once the barrier below has passed), so that the global
  // stores are 16 bytes per lane and whole contiguous rows per group of lanes (storing straight
  // from the accumulator arrangement, 32 bytes per row and instruction, measured slower).
  // Accumulator element e of block (i, j) is feature 16 i + 4 (l / 16) + e of token 16 j + l % 16.  Each
  // wavefront keeps its tile [WTOK tokens][16 MF features] in its own LDS region: rows of CPR 16-byte
  // chunks (8 features each), chunk position XORed with the row (16 rows at one logical chunk then cover
  // all banks, see eswz).  Only the wavefront itself touches the region: no barrier.
  constexpr int CPR = 2 * MF;                      // chunks per row
  constexpr int PITCH = CPR * 16;
  constexpr int RPI = 64 / CPR;                    // token rows per store instruction
  static_assert(4 * WTOK * PITCH <= (int)sizeof(PfShared<MF, TB>), "epilogue tile fits the stage buffers");
  unsigned char *E = smem_raw + wave_e * (WTOK * PITCH);
  // (256-byte rows span all banks; 128-byte rows half of them, the row's parity picks the half)
  auto eswz = [](int row) { return CPR == 16 ? (row & 15) : ((row >> 1) & (CPR - 1)); };
  // this lane's chunk: 8 consecutive features
  const int c = lane_e & (CPR - 1), rsub = lane_e / CPR;
  uint16_t *const out = Q.out;
  const long long ldo = Q.ldo;
  const int width = Q.width;
  const int col = (fb * BF_TILES + wf_e * MF) * 16 + c * 8;
  const bool lane_on = col < width;
  const bool wide = col + 8 <= width && ((reinterpret_cast<uintptr_t>(out) & 15u) == 0) && (ldo & 7) == 0;
  const int tok_base = tok0 + wt_e * WTOK + rsub;
  uint16_t *dst = out + (long long)tok_base * ldo + col;
  constexpr int NQ = WTOK / RPI;                   // store instructions per wavefront
  constexpr int NBATCH = (ROPE ? 8 : 4) * TB / 4, BQ = NQ / NBATCH;   // ... handled in batches (register budget)
  const bool lane_wide = lane_on && wide;
  constexpr int GR = 3;                            // table batches in registers: loads run two batches ahead
  // ROPE: this lane's 8 table values per row (cosines for the chunks of a head's first half, sines for
  // the others; the lane 8 further round the row of 16 lanes holds the other kind), two batches ahead
  // like the gate values.  All lanes load: the table row is clamped to the last token, never skipped.
  f32x4_t tab[GR][ROPE ? BQ : 1][2];
  auto load_tab = [&](int bt) {
    if constexpr (ROPE) {
      static_assert(!ROPE || CPR == 16, "one wavefront's features are one head of 128");
#pragma unroll
      for (int qq = 0; qq < BQ; ++qq) {
        const int tok = min(tok_base + (bt * BQ + qq) * RPI, P.T - 1);
        const float *tb = Q.rope + (long long)tok * 128 + (c & 7) * 8 + (c & 8) * 8;
        tab[bt % GR][qq][0] = *reinterpret_cast<const f32x4_t *>(tb);
        tab[bt % GR][qq][1] = *reinterpret_cast<const f32x4_t *>(tb + 4);
      }
    }
  };
  load_tab(0);
  __syncthreads();         // the epilogue reuses the LDS buffers (the loads above are in flight meanwhile)
  {
    const int wrow = lane_e & 15, wchunk = lane_e >> 5, whalf = ((lane_e >> 4) & 1) * 8;
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        uint2 w;
        if constexpr (GLU) {     // h = silu(gate) * up in fp32, one rounding of the result
          const uint2 sg = gpk[GLU ? i : 0][GLU ? j : 0];
          float u[4];            // (read out of the accumulator registers one by one, see the gate product above)
#pragma unroll
          for (int e = 0; e < 4; ++e) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(u[e]) : "a"(acc[i][j][e]));
          w.x = pack2<DT>(u[0] * lo_f32<DT>(sg.x), u[1] * hi_f32<DT>(sg.x));
          w.y = pack2<DT>(u[2] * lo_f32<DT>(sg.y), u[3] * hi_f32<DT>(sg.y));
        } else if constexpr (POST) {
          const uint2 b = bias[POST ? i : 0];
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[e]) : "a"(acc[i][j][e]));
          w.x = pack2<DT>(act_f32(v[0] + lo_f32<DT>(b.x), Q.post_act), act_f32(v[1] + hi_f32<DT>(b.x), Q.post_act));
          w.y = pack2<DT>(act_f32(v[2] + lo_f32<DT>(b.y), Q.post_act), act_f32(v[3] + hi_f32<DT>(b.y), Q.post_act));
        } else {
          w = pk[LATE ? 0 : i][LATE ? 0 : j];
        }
        // (the swizzle of row 16 j + wrow is that of wrow)
        *reinterpret_cast<uint2 *>(E + (16 * j + wrow) * PITCH + (((2 * i + wchunk) ^ eswz(wrow)) * 16) + whalf) = w;
        // (one pair at a time, in source order: scheduled freely, all 256 sums are read out of the
        // accumulator registers first, which does not fit beside the gate values)
        if constexpr (LATE) __builtin_amdgcn_sched_barrier(0);
      }
  }
  if (ROPE && NBATCH > 1) load_tab(1);
  // LDS reads of the next batch are issued before the stores of this one (different units)
  u32x4_t d[2][BQ];
  auto read_batch = [&](int bt, u32x4_t (&dd)[BQ]) {
#pragma unroll
    for (int qq = 0; qq < BQ; ++qq) {
      const int row = (bt * BQ + qq) * RPI + rsub;
      dd[qq] = *reinterpret_cast<const u32x4_t *>(E + row * PITCH + ((c ^ eswz(row)) * 16));
    }
  };
  auto store_batch = [&](int bt, u32x4_t (&dd)[BQ]) {
#pragma unroll
    for (int qq = 0; qq < BQ; ++qq) {
      const int q = bt * BQ + qq;
      if constexpr (ROPE) {
        // This lane's chunk c holds features 8 (c % 8) .. + 7 of the first (c < 8) or the second half
        // of a head, the lane 8 further round its row of 16 lanes holds the other element of each pair
        // and needs the same 8 angles: lanes c < 8 load the cosines, the others the sines, and the
        // values cross within the row (all lanes take part: the table row is clamped, not skipped).
        const f32x4_t m0 = tab[bt % GR][ROPE ? qq : 0][0], m1 = tab[bt % GR][ROPE ? qq : 0][1];
        const bool first = c < 8;
        u32x4_t r;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float mine_l = w < 2 ? m0[2 * w] : m1[2 * w - 4], mine_h = w < 2 ? m0[2 * w + 1] : m1[2 * w - 3];
          const float othr_l = across8(mine_l), othr_h = across8(mine_h);
          const uint32_t pw = across8(dd[qq][w]);                      // the partner elements
          const float cl = first ? mine_l : othr_l, ch = first ? mine_h : othr_h;
          const float sl = first ? -othr_l : mine_l, sh = first ? -othr_h : mine_h;   // a cos - b sin | b cos + a sin
          r[w] = pack2<DT>(lo_f32<DT>(dd[qq][w]) * cl + lo_f32<DT>(pw) * sl,
                           hi_f32<DT>(dd[qq][w]) * ch + hi_f32<DT>(pw) * sh);
        }
        dd[qq] = r;
      }
      if (lane_wide && tok_base + q * RPI < P.T)
        *reinterpret_cast<u32x4_t *>(dst + (long long)(q * RPI) * ldo) = dd[qq];
    }
  };
  read_batch(0, d[0]);
#pragma unroll
  for (int bt = 0; bt < NBATCH; ++bt) {
    if (ROPE && bt + 2 < NBATCH) load_tab(bt + 2);
    if (bt + 1 < NBATCH) read_batch(bt + 1, d[(bt + 1) & 1]);
    store_batch(bt, d[bt & 1]);
  }
  // Second copy of rank-space columns (t_k, t_v): this lane's chunk lies in one segment (whole 16-feature
  // tiles).  As a copy launch of its own (one element per thread) each of them read t back and took 19 us for
  // 8192 x 1228.  After the other stores, from the LDS tile once more: beside them it cost the plain kernels
  // registers that they do not have.
  if constexpr (!GLU && POSTK == PF_POST_NONE && !ROPE && !SPLIT) {
    uint16_t *dst2 = nullptr;
    long long ldo2 = 0;
    int n2 = 0;                                    // valid columns of the chunk in the second copy
#pragma unroll
    for (int g = 0; g < 3; ++g)
      if (g < Q.n_seg && lane_on && (col >> 4) >= Q.seg[g].tile0) {
        const int col2 = col - Q.seg[g].tile0 * 16;
        ldo2 = Q.seg[g].ldo2;
        n2 = Q.seg[g].out2 != nullptr ? Q.seg[g].width2 - col2 : 0;
        dst2 = Q.seg[g].out2 + (long long)tok_base * ldo2 + col2;
      }
    if (n2 > 0) {
#pragma unroll 4
      for (int q = 0; q < NQ; ++q) {
        if (tok_base + q * RPI >= P.T) break;
        const int row = q * RPI + rsub;
        const u32x4_t d = *reinterpret_cast<const u32x4_t *>(E + row * PITCH + ((c ^ eswz(row)) * 16));
        uint16_t *o = dst2 + (long long)(q * RPI) * ldo2;
        if (n2 >= 8) {
          *reinterpret_cast<u32x4_t *>(o) = d;
        } else {
#pragma unroll
          for (int e = 0; e < 7; ++e)
            if (e < n2) o[e] = (uint16_t)((d[e >> 1] >> ((e & 1) * 16)) & 0xffffu);
        }
      }
    }
  }
  // rare: output rows that are not 16-byte aligned, or the valid columns end inside this chunk
  if (lane_on && !wide) {
    for (int q = 0; q < NQ; ++q) {
      if (tok_base + q * RPI >= P.T) break;
      const int row = q * RPI + rsub;
      const u32x4_t d = *reinterpret_cast<const u32x4_t *>(E + row * PITCH + ((c ^ eswz(row)) * 16));
      uint16_t *o = dst + (long long)(q * RPI) * ldo;
      for (int e = 0; e < 8; ++e) {
        if (col + e >= width) break;
        unsigned v = (d[e >> 1] >> ((e & 1) * 16)) & 0xffffu;
        o[e] = (uint16_t)v;
      }
    }
  }
#else
  (void)P; (void)bid; (void)n_tiles; (void)n_tblocks; (void)fb_shift;
#endif
}

template <int DT, int MF, bool GLU, int POST = PF_POST_NONE, bool SPLIT = false, bool ROPE = false, int TB = 4>
__global__ __launch_bounds__(PF_THREADS) void prefill_kernel(const PfParams P) {
  prefill_body<DT, MF, GLU, POST, SPLIT, ROPE, TB>(P, (int)blockIdx.x, (int)gridDim.x, P.n_tblocks, 0);
}

// One launch with two tile shapes: the first P.n_big workgroups take 256 x 256 tiles of the feature
// blocks [0, P.fb_shift2), the others 128 x 256 tiles of the remaining feature blocks.  For large
// launches whose last round of 256 x 256 tiles would leave more than half of the compute units
// idle: that round's feature blocks run as twice as many smaller tiles, which take about 0.55 of a
// large tile's time each.
template <int DT, bool GLU, int POST, bool ROPE>
__global__ __launch_bounds__(PF_THREADS) void prefill_mixed_kernel(const PfParams P) {
  if ((int)blockIdx.x < P.n_big) prefill_body<DT, 8, GLU, POST, false, ROPE, 4>(P, (int)blockIdx.x, P.n_big, P.n_tblocks, 0);
  else prefill_body<DT, 8, GLU, POST, false, ROPE, 2>(P, (int)blockIdx.x - P.n_big, (int)gridDim.x - P.n_big, P.n_tblocks2, P.fb_shift2);
}

}  // namespace deinfer
