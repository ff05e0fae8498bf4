// Rank contraction over the rows of the permutation: for every row u of key q
//   out[u][r] = s_q * sum_c W_q[r][c] * src_u[c],   r < r_q,  s_q = alpha / r_q
// with either
//   src_u = x[row_token[u]]            (shared input; Sec. 3.5: once per row,
//                                       i.e. once per (token, active group))
//   src_u = S[t*k + j]                 (the row's single pair: per-pair input of
//                                       the down projection, or dY)
//   src_u = S[plist[u]]                (u a pair position: dY of that pair)
// and W = A (the shrink h = A_q x of Sec. 3.1.3) or W = B^T (dH = B_q^T dY).
// With out_w, the result of a single-pair row is multiplied by the pair's
// weight.
//
// Every sum is formed in a fixed order (deterministic).  Results go to any of
// three layouts:
//   row-major  [U][rpad]      operand of the expand kernel (zero beyond r_q)
//   per key    [R][ldh]       column u - offsets[q]: operand of the column pass
//   dense      [T*kslots][R]  per-token rows: operand of the dense dx GEMM
#include <type_traits>

#include "ace_device.hpp"
#include "ace_internal.hpp"

namespace ace {

namespace {

// Writes row u's result h (scaled, zero past r_q) to the requested outputs.
template <typename T, int RB>
__device__ inline void contract_store(const ContractArgs& a, int q, int lo, int u, f32x4 (&h)[RB]) {
  constexpr int KB = Tr<T>::KB, APF = Tr<T>::APF;
  const int k = a.k, R = a.keys.R;
  const int r_q = a.keys.rank[q], roff = a.keys.roff[q];
  const int nrb = ((r_q + KB - 1) / KB) * APF;
  const int g = (threadIdx.x & 63) >> 4;
  int tok = 0;
  uint32_t slots = 1u;
  if (a.src_mode != kSrcPairList) {
    tok = a.row_token[u];
    slots = a.row_slots[u];
  }
  if (a.out_w && a.pair_w) {  // single-pair rows: times the pair's weight
    const float w = a.pair_w[tok * k + (__builtin_ctz(slots | 0x80000000u) & 31)];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) h[rb] *= w;
  }
  if (a.out_row) {
    T* dst = static_cast<T*>(a.out_row) + (size_t)u * a.rpad;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int r0 = rank_of_row<T>(rb, 4 * g);  // 4 consecutive ranks
      if (r0 < a.rpad) {
#pragma unroll
        for (int v = 0; v < 4; ++v) dst[r0 + v] = (T)h[rb][v];
      }
    }
  }
  if (a.out_t && !a.out_t_pairs) {
    T* dst = static_cast<T*>(a.out_t);
    const long col = u - lo;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      if (rb < nrb) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = rank_of_row<T>(rb, 4 * g + v);
          if (r < r_q) dst[(size_t)(roff + r) * a.ldh + col] = (T)h[rb][v];
        }
      }
  }
  if (a.out_t && a.out_t_pairs) {  // one column per pair served, times its weight
    T* dst = static_cast<T*>(a.out_t);
    long col = a.ppos ? (long)a.ppos[u] - a.ppos[lo] : (long)(u - lo);
    for (uint32_t mm = slots; mm; mm &= mm - 1u, ++col) {
      const float w = a.pair_w ? a.pair_w[tok * k + __builtin_ctz(mm)] : 1.f;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        if (rb < nrb) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int r = rank_of_row<T>(rb, 4 * g + v);
            if (r < r_q) dst[(size_t)(roff + r) * a.ldh + col] = (T)(h[rb][v] * w);
          }
        }
    }
  }
  if (a.out_dense) {
    const int j0 = __builtin_ctz(slots | 0x80000000u) & 31;
    const size_t drow = (size_t)tok * a.kslots + (a.kslots > 1 ? j0 : 0);
    T* dst = static_cast<T*>(a.out_dense) + drow * R + roff;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      if (rb < nrb) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = rank_of_row<T>(rb, 4 * g + v);
          if (r < r_q) dst[r] = (T)h[rb][v];
        }
      }
  }
}

// ------------------------------------------------------------- small batches
//
// Few rows (decode batches): latency bounds a tile, not bytes.  A block of 8
// or 16 waves takes a tile of 16 rows; the waves split the contraction (wave w
// takes every NWV-th K-block), and each loads its fragments straight from
// global memory, up to SU K-blocks in flight, so that a contraction of 2048 is
// one or two round trips; the partial sums meet in LDS in wave order.
// OLMoE-like, 32 tokens, d_in 2048: 12.9 -> 9.4 us a call; fp32, 256 tokens,
// d_in 512 and 1024: 11.5 -> 8.8 and 15.2 -> 7.8 us.
// fp32, whose matrix work fills a tile, also takes larger batches this way, in
// tiles of 32 rows up to 128 ranks (launch_contract_f32).
// Tiles per grid row (a dimension holds fewer than 2^32 threads; a first tile
// passed as an argument is one more scalar load ahead of the tile search: 0.3
// of 8 us).
constexpr int kSmallGrid = 1 << 21;

// NRB row blocks of 16 per tile, NWV waves
template <int RB, int NRB_, int NWV_>
struct CSmall {
  static constexpr int NRB = NRB_, NWV = NWV_;
  static constexpr int SU = RB * NRB <= 4 ? 4 : RB * NRB <= 8 ? 2 : 1;   // K-blocks in flight per wave
  static constexpr int RRB = RB < 8 ? RB : 8;                // rank blocks per reduction pass
};

template <typename T, int RB, int NRB, int NWV>
__global__ __launch_bounds__(64 * NWV) void contract_small_kernel(ContractArgs a) {
  using F = typename Tr<T>::frag;
  using G = CSmall<RB, NRB, NWV>;
  constexpr int PER = Tr<T>::PER, KB = Tr<T>::KB, SU = G::SU;
  __shared__ f32x4 red[NWV][G::RRB][64];
  const int n_keys = a.keys.n_keys;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  int q, u0, u_end, lo;
  if (!locate_tile(a.offsets, n_keys, 16 * NRB, blockIdx.y * kSmallGrid + blockIdx.x, &q, &u0, &u_end,
                   a.src_mode == kSrcPairList ? a.ppos : nullptr, &lo))
    return;
  q = __builtin_amdgcn_readfirstlane(q);
  const int r_q = a.keys.rank[q], roff = a.keys.roff[q];
  const int nrb = (r_q + KB - 1) / KB * Tr<T>::APF;
  const int K = a.K, k = a.k;
  // rows past the segment repeat its last row and weight rows past r_q the
  // last one (never stored, zeroed before any store): every load is unconditional
  const T* srow[NRB];
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib) {
    const int uc = min(u0 + 16 * ib + c16, u_end - 1);
    int sr;
    if (a.src_mode == kSrcPairList) {
      sr = a.plist[uc];
    } else {
      const int tok = a.row_token[uc];
      const uint32_t sl = a.row_slots[uc];
      sr = a.src_mode == kSrcPerPair ? tok * k + (__builtin_ctz(sl | 0x80000000u) & 31) : tok;
    }
    srow[ib] = static_cast<const T*>(a.src) + (size_t)sr * K;
  }
  const T* wrow[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int r = rank_of_row<T>(rb, c16);
    wrow[rb] = static_cast<const T*>(a.W) + (size_t)(roff + min(r, r_q - 1)) * a.ldw;
  }
  f32x4 acc[NRB][RB];
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[ib][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nks = (K + KB - 1) / KB;
  for (int ks = wave; ks < nks; ks += NWV * SU) {
    F sf[SU][NRB], wf[SU][RB];
    // chunks past the end repeat the row's last one, zeroed below (both
    // operands: an infinity there must not meet a zero)
#pragma unroll
    for (int s = 0; s < SU; ++s) {
      const int kof = (ks + NWV * s) * KB + PER * g, kc = min(kof, K - PER);
#pragma unroll
      for (int ib = 0; ib < NRB; ++ib) sf[s][ib] = Tr<T>::load(srow[ib] + kc);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        if (rb < nrb) wf[s][rb] = Tr<T>::load(wrow[rb] + kc);
    }
#pragma unroll
    for (int s = 0; s < SU; ++s) {
      const int kof = (ks + NWV * s) * KB + PER * g;
      if (ks + NWV * s < nks) {
#pragma unroll
        for (int ib = 0; ib < NRB; ++ib) {
          if (kof >= K) sf[s][ib] = Tr<T>::zero();
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            if (kof >= K) wf[s][rb] = Tr<T>::zero();
            if (rb < nrb) acc[ib][rb] = Tr<T>::mma(wf[s][rb], sf[s][ib], acc[ib][rb]);
          }
        }
      }
    }
  }
  // partial sums, added in wave order; wave 0 finishes the rows
  const float s = a.alpha / (float)r_q;
  f32x4 h[NRB][RB];
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib)
#pragma unroll
    for (int p = 0; p < RB / G::RRB; ++p) {
      if (ib + p > 0) __syncthreads();
#pragma unroll
      for (int rb = 0; rb < G::RRB; ++rb) red[wave][rb][lane] = acc[ib][p * G::RRB + rb];
      __syncthreads();
      // wave w sums rank block w's partials
      if (wave < G::RRB) {
        f32x4 t = red[0][wave][lane];
#pragma unroll
        for (int w = 1; w < NWV; ++w) t += red[w][wave][lane];
        red[0][wave][lane] = t;
      }
      __syncthreads();
      if (wave == 0) {
#pragma unroll
        for (int rb = 0; rb < G::RRB; ++rb) h[ib][p * G::RRB + rb] = red[0][rb][lane] * s;
      }
    }
  if (wave != 0) return;
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib) {
    const int u = u0 + 16 * ib + c16;
    if (u >= u_end) continue;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (rank_of_row<T>(rb, 4 * g + v) >= r_q) h[ib][rb][v] = 0.f;
    contract_store<T, RB>(a, q, lo, u, h[ib]);
  }
}

// ------------------------------------------------------- fp32, larger batches
//
// A block of four waves takes a tile of 64 rows (32 from 65 ranks); the waves
// split the contraction and keep the next K-blocks' fragments in flight in
// registers, so the weights are read half as often as by 32-row tiles (the
// same at 32) and no K-block waits for its loads; the partial sums meet in
// LDS in a fixed order.  Every sum is four chains of a quarter of the
// contraction.  Tiles go to the XCDs by token range, as in contract_dma.
template <int RB>
struct CReg {
  static constexpr int NRB = RB <= 4 ? 4 : 2;   // 16-row blocks per tile
  static constexpr int UNROLL = 2;             // K-blocks per stage
};

template <int RB>
__global__ __launch_bounds__(kThreads) void contract_reg_kernel(ContractArgs a) {
  using T = float;
  using F = typename Tr<T>::frag;
  constexpr int PER = Tr<T>::PER, KB = Tr<T>::KB, APF = Tr<T>::APF;
  constexpr int NRB = CReg<RB>::NRB, U = CReg<RB>::UNROLL;
  constexpr int BM = 16 * NRB;
  __shared__ int seg[kMaxKeys + 1];
  __shared__ int bstart[kMaxKeys + 1];
  __shared__ int bfirst[kMaxKeys];
  __shared__ int scan[kThreads];
  __shared__ f32x4 red[4][NRB][RB][64];
  const int n_keys = a.keys.n_keys;
  const int bucket = blockIdx.x % kXcds;
  build_bucket_table(a.offsets, a.src_mode == kSrcPairList ? a.ppos : nullptr, n_keys, BM, bucket,
                     seg, bstart, bfirst, scan);
  const int total = bstart[n_keys];
  const int stride = gridDim.x / kXcds;  // the grid is a multiple of kXcds
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c16 = lane & 15, g = lane >> 4;
  const T* S = static_cast<const T*>(a.src);
  const T* W = static_cast<const T*>(a.W);
  const int K = a.K, k = a.k;
  const int nks = (K + KB - 1) / KB, nks_full = K / KB;

  for (int idx = blockIdx.x / kXcds; idx < total; idx += stride) {
    const int q = upper_index(bstart, n_keys, idx);
    const int lo = seg[q];
    const int u0 = lo + (bfirst[q] + idx - bstart[q]) * BM;
    const int u_end = seg[q + 1];
    const int r_q = a.keys.rank[q], roff = a.keys.roff[q];
    const int nmb = (r_q + KB - 1) / KB;
    const int nrb = nmb * APF;  // rank blocks spanned by rank_of_row for r < r_q

    // Source rows.  Rows past the segment re-read the last row (never
    // stored); weight rows past r_q re-read row r_q - 1 (zeroed before any
    // store), so every load is unconditional and a wave keeps all of them in
    // flight.
    const T* srow[NRB];
    int sv[NRB];
    uint32_t slv[NRB];
#pragma unroll
    for (int ib = 0; ib < NRB; ++ib) {  // unconditional loads: one round trip
      const int uc = min(u0 + 16 * ib + c16, u_end - 1);
      if (a.src_mode == kSrcPairList) {
        sv[ib] = a.plist[uc];
        slv[ib] = 1u;
      } else {
        sv[ib] = a.row_token[uc];
        slv[ib] = a.row_slots[uc];
      }
    }
#pragma unroll
    for (int ib = 0; ib < NRB; ++ib) {
      const int j0 = __builtin_ctz(slv[ib] | 0x80000000u) & 31;
      const int sr = a.src_mode == kSrcPerPair ? sv[ib] * k + j0 : sv[ib];
      srow[ib] = S + (size_t)sr * K;
    }
    const T* wrow[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int r = rank_of_row<T>(rb, c16);
      wrow[rb] = W + (size_t)(roff + (r < r_q ? r : r_q - 1)) * a.ldw;
    }

    f32x4 acc[NRB][RB];
#pragma unroll
    for (int ib = 0; ib < NRB; ++ib)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) acc[ib][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Main loop over this wave's full stages (U K-blocks each), register
    // double-buffered: the next stage's loads are in flight while the
    // matrix cores work on the current one.
    struct Stage {
      F sf[U][NRB];
      F wf[U][RB];
    };
    auto load_stage = [&](int ks0, Stage& st) {
#pragma unroll
      for (int s = 0; s < U; ++s) {
        const int kof = (ks0 + 4 * s) * KB + PER * g;
#pragma unroll
        for (int ib = 0; ib < NRB; ++ib) st.sf[s][ib] = Tr<T>::load(srow[ib] + kof);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) st.wf[s][rb] = Tr<T>::load(wrow[rb] + kof);
      }
    };
    auto mma_stage = [&](const Stage& st) {
#pragma unroll
      for (int s = 0; s < U; ++s)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
          if (rb < nrb) {
#pragma unroll
            for (int ib = 0; ib < NRB; ++ib) acc[ib][rb] = Tr<T>::mma(st.wf[s][rb], st.sf[s][ib], acc[ib][rb]);
          }
    };
    // stages of this wave: ks0 = wave + 4*U*i with ks0 + 4*(U-1) < nks_full
    const int n_main = nks_full > wave + 4 * (U - 1) ? (nks_full - wave - 4 * (U - 1) + 4 * U - 1) / (4 * U) : 0;
    {
      Stage SA, SB;
      if (n_main > 0) load_stage(wave, SA);
      int i = 0;
      for (; i + 1 < n_main; i += 2) {
        load_stage(wave + 4 * U * (i + 1), SB);
        mma_stage(SA);
        if (i + 2 < n_main) load_stage(wave + 4 * U * (i + 2), SA);
        mma_stage(SB);
      }
      if (i < n_main) mma_stage(SA);
    }
    int ks0 = wave + 4 * U * n_main;
    for (; ks0 < nks; ks0 += 4) {  // leftover K-blocks of this wave (masked tail)
      const int kof = ks0 * KB + PER * g;
      const int nv = K - kof;
      const int kc = nv > 0 ? kof : 0;
      F sf[NRB], wf[RB];
#pragma unroll
      for (int ib = 0; ib < NRB; ++ib) sf[ib] = nv > 0 ? load_frag<T>(srow[ib] + kc, nv, true) : Tr<T>::zero();
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) wf[rb] = load_frag<T>(wrow[rb] + kc, nv, true);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        if (rb < nrb) {
#pragma unroll
          for (int ib = 0; ib < NRB; ++ib) acc[ib][rb] = Tr<T>::mma(wf[rb], sf[ib], acc[ib][rb]);
        }
    }

    // ---- partial sums meet in LDS; wave w finishes row block w % NRB
    __syncthreads();
#pragma unroll
    for (int ib = 0; ib < NRB; ++ib)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) red[wave][ib][rb][lane] = acc[ib][rb];
    __syncthreads();
    const int ib = wave % NRB;
    if (wave >= NRB) continue;  // the other waves' row blocks are done by waves < NRB
    const int u = u0 + 16 * ib + c16;
    if (u0 + 16 * ib >= u_end) continue;  // wave-uniform
    const bool valid = u < u_end;
    const float s = a.alpha / (float)r_q;
    f32x4 h[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      h[rb] = (((red[0][ib][rb][lane] + red[1][ib][rb][lane]) + red[2][ib][rb][lane]) +
               red[3][ib][rb][lane]) * s;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (rank_of_row<T>(rb, 4 * g + v) >= r_q) h[rb][v] = 0.f;
    }
    if (!valid) continue;
    contract_store<T, RB>(a, q, lo, u, h);
  }
}

// ------------------------------------------------------- bf16, larger batches
//
// A block takes a tile of 64 rows of one key; wave w owns rows 16w .. 16w+15
// for every rank over the whole contraction, so no cross-wave reduction is
// needed.  Stages of KC contraction indices of the 64 source rows and of the
// key's weight rows are copied global -> LDS (global_load_lds_dwordx4, row
// pieces with 16-byte chunks XOR-swizzled by row), NBUF stages in flight;
// MFMA fragments are plain 16-byte LDS reads.  Only the weight rows below r_q
// (rounded up to a copy) are copied.
//
// Row sums (row_sum, pair-position sources): a row serves up to k pairs, at
// consecutive positions.  A tile then takes the rows whose first pair lies in
// a window of 65 - k positions, so their pairs (at most 64) are all in the
// tile; the per-pair results times the pair weights go to LDS in fp32 and
// every row's sum (pairs in position order) is stored once.
//
// DEEP: with no more tiles than CUs (decode batches) a block is alone on its
// CU and every stage would cost a round trip to memory: the stages fill the
// LDS instead of sharing it with other blocks, a block takes one tile, found
// without barriers.  OLMoE-like, 1000 tokens (189 tiles at most): a pass of
// the three adapters 96 -> 86 us.
template <int RB, int NWV, bool DEEP>
struct CDma {
  // bytes of a row per stage and stages in LDS: ranks up to 32 take 256-byte
  // stages two deep (three blocks per CU); larger ranks, whose weight rows
  // double the bytes of a stage, 128-byte stages three deep
  static constexpr int ROWB = RB <= 2 || (DEEP && RB == 4) ? 256 : 128;
  static constexpr int NBUF = DEEP ? (RB == 4 ? 4 : 6) : ROWB == 256 ? 2 : 3;
  static constexpr int KC = ROWB / 2;            // contraction indices per stage
  static constexpr int THREADS = 64 * NWV;       // NWV waves of 16 tile rows each
  static constexpr int ROWS = 16 * NWV;          // tile rows
  static constexpr int CPR = ROWB / 16;          // 16-byte chunks per row piece
  static constexpr int RPI = 64 / CPR;           // row pieces per copy instruction
  static constexpr int SBYTES = ROWS * ROWB;     // tile source rows
  static constexpr int WROWS = 16 * RB;
  static constexpr int WBYTES = WROWS * ROWB;    // weight rows
  static constexpr int NS = 16 / RPI;            // source copies per wave per stage
  static constexpr int NW = (WROWS / RPI + NWV - 1) / NWV;   // weight copies per wave per stage (at most)
  static constexpr int LDS = NBUF * (SBYTES + WBYTES);
  // LDS per CU is 160 KiB; the tile tables take about 4 KiB more per block
  static constexpr int BLOCKS_PER_CU = (160 * 1024) / (LDS + 4 * 1024 + 512) < 1 ? 1 : (160 * 1024) / (LDS + 4 * 1024 + 512);
  // row sums: per-pair results [ROWS][RPS] fp32 over the stage buffers
  static constexpr int RPS = 16 * RB + 4;   // 16-byte skew between positions
  static_assert(ROWS * RPS * 4 <= LDS, "per-pair results exceed the stage buffers");
  static_assert(WROWS / RPI <= NWV * NW, "weight copies");
  static_assert((NBUF - 2) * (NS + NW) < 64, "copies in flight per wave");
};

// Chunk swizzle of weight row w (CPR 16-byte chunks per staged row).  A
// fragment read touches the rows rank_of_row(rb, i), i = 0..15: w & 3 = i & 3,
// bit 2 of w = rb & 1 and bits 3.. = i >> 2, so w & (CPR - 1) alone would give
// only four distinct chunk positions among the first eight lanes at 8 chunks
// per row (two-way bank conflicts); folding bit 3 into bit 2 spreads them
// over eight (and the 16 rows over 16 positions at 16 chunks per row).
template <int CPR>
__device__ inline int w_swz(int w) { return (w ^ ((w >> 3) << 2)) & (CPR - 1); }

// Tile size in pair positions when rows are summed (every row's pairs lie in
// the tile) or rows otherwise, for tiles of `rows` rows.
inline __host__ __device__ int contract_tile(int row_sum, int k, int rows) {
  return row_sum ? rows + 1 - k : rows;
}

// Row sums of a tile whose pair positions p0 .. p1 - 1 hold rows ua .. ub - 1
// (rstart = first position of this lane's row ua + 64 (wave / 4) + lane, rend
// the next row's, rtok its token): the per-pair results, scaled and times the
// pair weights, go to LDS (fp32); then lane l of wave w sums row ua + 64 (w /
// 4) + l over its pairs in position order for the rank chunks 8 (w % 4),
// 8 (w % 4) + 32, ... and stores the bf16 sum per key (column u - rfirst)
// and/or per token.
template <int RB, int NWV, bool DEEP>
__device__ inline void row_sum_store(const ContractArgs& a, int q, const f32x4 (&acc)[RB], float s,
                                     float pw, int ua, int ub, int p0, int rfirst, int rstart,
                                     int rend, int rtok, float* hp) {
  constexpr int RPS = CDma<RB, NWV, DEEP>::RPS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c16 = lane & 15, g = lane >> 4;
  const int r_q = a.keys.rank[q], roff = a.keys.roff[q], R = a.keys.R;
  __syncthreads();   // every wave is done reading the staging buffers
  {
    float* dst = hp + (16 * wave + c16) * RPS;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int r0 = rank_of_row<__bf16>(rb, 4 * g);   // 4 consecutive ranks
      f32x4 h = (acc[rb] * s) * pw;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (r0 + v >= r_q) h[v] = 0.f;
      *reinterpret_cast<f32x4*>(dst + r0) = h;
    }
  }
  __syncthreads();
  const int u = ua + 64 * (wave / 4) + lane;
  if (u >= ub) return;
  const int b0 = rstart - p0, b1 = rend - p0;
  __bf16* dt = static_cast<__bf16*>(a.out_t);
  const long col = u - rfirst;
  __bf16* df = a.out_dense ? static_cast<__bf16*>(a.out_dense) + (size_t)rtok * R + roff : nullptr;
  for (int r0 = 8 * (wave % 4); r0 < r_q; r0 += 32) {
    const float* src = hp + b0 * RPS + r0;
    f32x4 lo = *reinterpret_cast<const f32x4*>(src), hi = *reinterpret_cast<const f32x4*>(src + 4);
    for (int pos = b0 + 1; pos < b1; ++pos) {
      src += RPS;
      lo += *reinterpret_cast<const f32x4*>(src);
      hi += *reinterpret_cast<const f32x4*>(src + 4);
    }
    const bf16x8 v = {(__bf16)lo[0], (__bf16)lo[1], (__bf16)lo[2], (__bf16)lo[3],
                      (__bf16)hi[0], (__bf16)hi[1], (__bf16)hi[2], (__bf16)hi[3]};
    if (dt) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (r0 + e < r_q) dt[(size_t)(roff + r0 + e) * a.ldh + col] = v[e];
    }
    if (df) {
      if (r0 + 8 <= r_q && (((roff + r0) | R) & 7) == 0) {   // 16-byte aligned in every token's row
        Tr<__bf16>::store(df + r0, v);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (r0 + e < r_q) df[r0 + e] = v[e];
      }
    }
  }
}

template <int RB, int NWV, bool DEEP>
__global__ __launch_bounds__(64 * NWV, RB == 8 && !DEEP ? 2 : 1) void contract_dma_kernel(ContractArgs a) {
  using T = __bf16;
  using G = CDma<RB, NWV, DEEP>;
  using F = typename Tr<T>::frag;
  constexpr int KC = G::KC, NBUF = G::NBUF, KB = Tr<T>::KB, PER = Tr<T>::PER, ROWB = G::ROWB;
  constexpr int CPR = G::CPR, RPI = G::RPI;
  // stage buffers: NBUF source stages, then NBUF weight stages; the row sums
  // reuse the whole area for the per-pair results
  __shared__ __attribute__((aligned(16))) char smem[G::LDS];
  char (*Sb)[G::SBYTES] = reinterpret_cast<char (*)[G::SBYTES]>(smem);
  char (*Wb)[G::WBYTES] = reinterpret_cast<char (*)[G::WBYTES]>(smem + NBUF * G::SBYTES);
  constexpr int TAB = DEEP ? 1 : kMaxKeys + 1;   // tile tables
  __shared__ int seg[TAB];
  __shared__ int bstart[TAB];
  __shared__ int bfirst[TAB];
  __shared__ int scan[DEEP ? 1 : kThreads];   // block_exclusive_scan reads the first kThreads / 64
  static_assert(G::THREADS >= kMaxKeys, "one thread per key in the tile tables");
  const int n_keys = a.keys.n_keys;
  const int bucket = blockIdx.x % kXcds;
  const int K = a.K, k = a.k;
  const bool rsum = a.row_sum != 0;   // implies kSrcPairList
  const int TS = contract_tile(a.row_sum, k, G::ROWS);
  const int32_t* seg_map = a.src_mode == kSrcPairList ? a.ppos : nullptr;
  int total = 1, stride = 1;
  if constexpr (!DEEP) {
    build_bucket_table(a.offsets, seg_map, n_keys, TS, bucket, seg, bstart, bfirst, scan);
    total = bstart[n_keys];
    stride = gridDim.x / kXcds;  // the grid is a multiple of kXcds
  }
  // wave-uniform values kept in scalar registers (uniform branches, no exec masks)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  const T* S = static_cast<const T*>(a.src);
  const T* W = static_cast<const T*>(a.W);
  const int cpos = lane & (CPR - 1), crow = lane / CPR;   // 16-byte position / row inside a copy

  for (int idx = DEEP ? 0 : blockIdx.x / kXcds; idx < total; idx += stride) {
    const int nst = (K + KC - 1) / KC;
    int q, lo, u0, u_end;
    if constexpr (DEEP) {
      if (!locate_tile(a.offsets, n_keys, TS, blockIdx.x, &q, &u0, &u_end, seg_map, &lo)) return;
      q = __builtin_amdgcn_readfirstlane(q);
    } else {
      q = upper_index(bstart, n_keys, idx);
      lo = seg[q];
      u0 = lo + (bfirst[q] + idx - bstart[q]) * TS;
      u_end = seg[q + 1];
    }
    const int r_q = a.keys.rank[q], roff = a.keys.roff[q];
    // row sums: rows ua .. ub - 1 start inside the window [u0, u0 + TS); their
    // pairs are positions ppos[ua] .. ppos[ub] - 1, which become u0 .. u_end
    int ua = 0, ub = 0, rfirst = 0, rtok = 0, rstart = 0, rend = 0;
    float pw = 1.f;
    if (rsum) {
      const int y = (lane & 1) ? min(u0 + TS, u_end) : u0;
      int row, pos;
      if (y < u_end) {   // first row starting at or after position y
        const int r0 = a.pair_row[a.plist[y]];
        const int s0 = a.ppos[r0], s1 = a.ppos[r0 + 1];
        row = s0 == y ? r0 : r0 + 1;
        pos = s0 == y ? s0 : s1;
      } else {
        row = a.offsets[q + 1];
        pos = u_end;
      }
      ua = __shfl(row, 0);
      ub = __shfl(row, 1);
      u0 = __shfl(pos, 0);
      u_end = __shfl(pos, 1);
      if (ua >= ub) continue;   // block-uniform: no row starts in this window
      rfirst = a.offsets[q];
      const int er = ua + 64 * (wave / 4) + lane;   // this lane's row in the epilogue
      if (er < ub) {
        rstart = a.ppos[er];
        rend = er + 1 < ub ? a.ppos[er + 1] : u_end;
        rtok = a.row_token[er];
      }
      if (a.pair_w) pw = a.pair_w[a.plist[min(u0 + 16 * wave + c16, u_end - 1)]];
    }
    // weight copies this wave issues per stage (rows below r_q only)
    const int wcopies = (r_q + RPI - 1) / RPI;
    const int nw = min(G::NW, max(0, wcopies - wave * G::NW));
    // source copies: with DEEP none for rows past the segment (their results
    // are not stored); otherwise those repeat the last row, since a branch per
    // copy slows full tiles
    const int ns = DEEP ? __builtin_amdgcn_readfirstlane(
                              min(G::NS, max(0, (u_end - u0 - 16 * wave + RPI - 1) / RPI)))
                        : G::NS;

    // source rows this lane copies (rows past the segment re-read the last
    // one) and the chunk of the row piece it copies
    const T* sptr[G::NS];
    int scol[G::NS];
#pragma unroll
    for (int i = 0; i < G::NS; ++i) {
      const int uc = min(u0 + 16 * wave + RPI * i + crow, u_end - 1);
      int sr;
      if (a.src_mode == kSrcPairList) {
        sr = a.plist[uc];
      } else {
        const int tok = a.row_token[uc];
        sr = a.src_mode == kSrcPerPair ? tok * k + (__builtin_ctz(a.row_slots[uc] | 0x80000000u) & 31) : tok;
      }
      sptr[i] = S + (size_t)sr * K;
      scol[i] = PER * (cpos ^ ((16 * wave + RPI * i + crow) & (CPR - 1)));
    }
    const T* wptr[G::NW];
    int wcol[G::NW];
#pragma unroll
    for (int i = 0; i < G::NW; ++i) {
      const int rl = RPI * (wave * G::NW + i) + crow;  // weight row of the tile (rank)
      wptr[i] = W + (size_t)(roff + min(rl, r_q - 1)) * a.ldw;
      wcol[i] = PER * (cpos ^ w_swz<CPR>(rl));
    }
    // copies of stage st (columns past K are clamped; masked at the reads)
    auto issue = [&](int st) {
      const int b = st % NBUF;
      const int k0 = st * KC;
#pragma unroll
      for (int i = 0; i < G::NS; ++i)
        if (i < ns)
          dma16(sptr[i] + min(k0 + scol[i], K - PER),
                __builtin_amdgcn_readfirstlane(lds_addr(&Sb[b][(16 * wave + RPI * i) * ROWB])));
#pragma unroll
      for (int i = 0; i < G::NW; ++i)
        if (i < nw)
          dma16(wptr[i] + min(k0 + wcol[i], K - PER),
                __builtin_amdgcn_readfirstlane(lds_addr(&Wb[b][RPI * (wave * G::NW + i) * ROWB])));
    };
    const int per_stage = ns + nw;   // copies per stage of this wave

    __syncthreads();  // the previous tile is done with the buffers
    f32x4 acc[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < NBUF - 1; ++p)
      if (p < nst) issue(p);
    // this wave's copies of stage st are done once at most those of the
    // stages issued after it are outstanding; the barrier publishes them
    auto begin_stage = [&](int st) {
      wait_vmcnt_upto<(NBUF - 2) * (G::NS + G::NW)>(min(NBUF - 2, nst - 1 - st) * per_stage);
      __syncthreads();
      if (st + NBUF - 1 < nst) issue(st + NBUF - 1);
    };
    // K-block kb of stage st; the ragged form zeroes the fragments past the
    // contraction (whole ones: K is a multiple of a chunk), both operands, so
    // that an infinity there does not meet a zero
    auto kblock = [&](int st, int kb, bool ragged) {
      const int b = st % NBUF;
      const int kk = st * KC + kb * KB;
      const int chunk = kb * 4 + g;
      const int rl = 16 * wave + c16;
      F sf = *reinterpret_cast<const F*>(&Sb[b][rl * ROWB + ((chunk ^ (rl & (CPR - 1))) << 4)]);
      const bool past = ragged && kk + PER * g >= K;
      if (past) sf = Tr<T>::zero();
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        // weight rows at or past r_q were not copied: their results are zeroed below
        const int wr = rank_of_row<T>(rb, c16);
        F wf = *reinterpret_cast<const F*>(&Wb[b][wr * ROWB + ((chunk ^ w_swz<CPR>(wr)) << 4)]);
        if (past) wf = Tr<T>::zero();
        acc[rb] = Tr<T>::mma(wf, sf, acc[rb]);   // D[rank][row]
      }
    };
    // full stages: a loop with no branch around the matrix work (a branch
    // there made the compiler copy the accumulators every stage)
    const int nst_full = K / KC;
    for (int st = 0; st < nst_full; ++st) {
      begin_stage(st);
#pragma unroll
      for (int kb = 0; kb < KC / KB; ++kb) kblock(st, kb, false);
    }
    if (nst_full < nst) {   // block-uniform: the last, partial stage
      const int st = nst_full;
      begin_stage(st);
#pragma unroll
      for (int kb = 0; kb < KC / KB; ++kb) {
        const int kk = st * KC + kb * KB;
        if (kk < K) kblock(st, kb, kk + KB > K);
      }
    }

    const float s = a.alpha / (float)r_q;
    if (rsum) {
      row_sum_store<RB, NWV, DEEP>(a, q, acc, s, pw, ua, ub, u0, rfirst, rstart, rend, rtok,
                             reinterpret_cast<float*>(smem));
      continue;
    }
    const int u = u0 + 16 * wave + c16;
    if (u0 + 16 * wave >= u_end || u >= u_end) continue;
    f32x4 h[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      h[rb] = acc[rb] * s;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (rank_of_row<T>(rb, 4 * g + v) >= r_q) h[rb][v] = 0.f;
    }
    contract_store<T, RB>(a, q, lo, u, h);
  }
}

// Tiles of BM rows, at most.
long max_tiles(const ContractArgs& a, long P, int BM) { return P > 0 ? (P + BM - 1) / BM + a.keys.n_keys : 0; }

template <typename T, int RB, int NRB, int NWV>
hipError_t launch_small(const ContractArgs& a, long P, hipStream_t stream) {
  const long n = max_tiles(a, P, 16 * NRB);
  const dim3 grid((unsigned)(n < kSmallGrid ? n : kSmallGrid), (unsigned)((n + kSmallGrid - 1) / kSmallGrid));
  if (n > 0) contract_small_kernel<T, RB, NRB, NWV><<<grid, 64 * NWV, 0, stream>>>(a);
  return hipGetLastError();
}

// Tiles of 16 rows (at most) up to which small batches go to contract_small:
// above, the tiles re-read the weights too often (1000 tokens, 564 tiles: a
// pass of the three adapters takes 105 us with it, 86 without; 400 tokens, 216
// tiles: 67 against 71).
constexpr long kSmallTiles = 256;

// bf16: sixteen waves from 128 K-blocks (4096 indices), eight below, where a
// wave's share is a few K-blocks and the reduction over the waves weighs more:
// rank 48, d_in 512 17.2 against 13.0 us a forward call (the LDS-staged kernel
// 15.2), d_in 2048 17.5 and 17.3, d_in 8192 43.7 and 46.2.  fp32 sums in
// sixteen chains throughout: eight are 1.4 us of 56 a tiny training step
// faster, and off by 2.9e-7 from 64 bits where sixteen are by 2.5e-7.  Above
// 128 ranks eight (at sixteen the registers spill).
template <typename T, int RB>
hipError_t launch_few_rows(const ContractArgs& a, long P, hipStream_t stream) {
  if constexpr (RB <= 8)
    if (std::is_same<T, float>::value || (a.K + Tr<T>::KB - 1) / Tr<T>::KB >= 128)
      return launch_small<T, RB, 1, 16>(a, P, stream);
  return launch_small<T, RB, 1, 8>(a, P, stream);
}

template <int RB>
hipError_t launch_contract_bf16(const ContractArgs& a, long P, hipStream_t stream) {
  constexpr int NWV = 4;
  using G = CDma<RB, NWV, false>;
  if (!a.row_sum && max_tiles(a, P, 16) <= kSmallTiles) return launch_few_rows<__bf16, RB>(a, P, stream);
  const long tiles = max_tiles(a, P, contract_tile(a.row_sum, a.k, G::ROWS));
  if constexpr (RB <= 8) {
    // one block per CU and one tile per block: see DEEP
    if (tiles > 0 && tiles <= device_cu_count()) {
      contract_dma_kernel<RB, NWV, true><<<(int)tiles, G::THREADS, 0, stream>>>(a);
      return hipGetLastError();
    }
  }
  // tiles per bucket <= (all tiles) / kXcds + n_keys
  const long pb = P > 0 ? tiles / kXcds + a.keys.n_keys : 0;
  const long cap = (long)G::BLOCKS_PER_CU * device_cu_count() / kXcds;
  const int grid = (int)(pb < cap ? pb : cap) * kXcds;
  if (grid > 0) contract_dma_kernel<RB, NWV, false><<<grid, G::THREADS, 0, stream>>>(a);
  return hipGetLastError();
}

template <int RB>
hipError_t launch_contract_reg(const ContractArgs& a, long P, hipStream_t stream) {
  // tiles per bucket <= (all tiles) / kXcds + n_keys
  const long pb = max_tiles(a, P, 16 * CReg<RB>::NRB) / kXcds + a.keys.n_keys;
  const long cap = 6L * device_cu_count() / kXcds;
  contract_reg_kernel<RB><<<(int)(pb < cap ? pb : cap) * kXcds, kThreads, 0, stream>>>(a);
  return hipGetLastError();
}

// Beyond the small batches, contract_small in tiles of 32 rows (16 above 128
// ranks) or contract_reg.  Its buckets need several tiles per key to be even
// (64 keys of 128 pairs, rank 100, d_in 2048: 139 us with it, 67 without), and
// there:
//   ranks 65..128   from 1024 indices (4096 pairs through 8 keys, d_in 1024,
//                   4096 and 14336: 41 / 43, 93 / 108, 267 / 314 us; d_in 512,
//                   16,384 pairs: 76 / 72)
//   ranks up to 64  where its tiles, twice as large, take half the rounds of
//                   blocks: contract_reg / contract_small at d_in 2048 and 8192,
//                   8 keys, rank 32 12,000 rows 35 / 44 and 97 / 127; 16,000, two
//                   rounds of both, 66 / 46 and 223 / 129; rank 64 53 / 66 and
//                   152 / 197, 95 / 69 and 291 / 202; 32,000, two and four, 107 /
//                   127 and 319 / 424 (rank 32 74 / 76 and 240 / 251: one round
//                   only up to there); and from three rounds on at ranks above
//                   32 and 4096 indices (65,536 pairs, d_in 4096 402 / 437, 14336
//                   1239 / 1519; d_in 2048 230 / 231)
// contract_reg's tiles are dealt to the XCDs key by key, so its rounds are
// counted with half a tile per key and XCD more than the rows fill (15 keys of
// 2133 rows, 508 tiles, took three rounds).  Rows that serve several slots are
// fewer than pairs, at most one per token and key; how many fewer the routing
// decides (7% with 15 even keys of four experts, top 4), so either kernel's
// rounds are counted on the safe side.
// Above 128 ranks contract_small is ahead throughout (rank 200, d_in 2048,
// 4096 to 32,768 pairs through 8 keys: 135 to 564 against 143 to 592).
template <int RB>
hipError_t launch_contract_f32(const ContractArgs& a, long P, hipStream_t stream) {
  if constexpr (RB > 8) {
    return launch_small<float, RB, 1, 8>(a, P, stream);
  } else {
    if (max_tiles(a, P, 16) <= kSmallTiles) return launch_few_rows<float, RB>(a, P, stream);
    const long keys = a.keys.n_keys, cus = device_cu_count();
    if constexpr (RB == 8) {
      if (a.K >= 1024 && P >= 256 * keys) return launch_contract_reg<RB>(a, P, stream);
      return launch_small<float, RB, 2, 8>(a, P, stream);
    } else {
      const long most = a.multi_slot && P / a.k * keys < P ? P / a.k * keys : P;
      const long r64 = (most / 64 + 4 * keys + cus - 1) / cus;
      const long r32 = ((a.multi_slot ? most * 3 / 4 : most) / 32 + cus - 1) / cus;
      if (P >= 512 * keys && ((r32 >= 2 * r64 && (RB == 4 || r64 == 1)) ||
                              (RB == 4 && a.K >= 4096 && r64 >= 3)))
        return launch_contract_reg<RB>(a, P, stream);
      return launch_small<float, RB, 2, 4>(a, P, stream);
    }
  }
}

}  // namespace

int rank_blocks(int r_max) {
  const int rb = (r_max + 15) / 16;
  return rb <= 2 ? 2 : rb <= 4 ? 4 : rb <= 8 ? 8 : 16;
}

int rank_pad(int dtype, int r_max) {
  // KB * (RB / APF) = 16 * RB for both element types
  (void)dtype;
  return 16 * rank_blocks(r_max);
}

hipError_t launch_contract(int dtype, const ContractArgs& a, int r_max, long P,
                           hipStream_t stream) {
  if (a.row_sum && (dtype != ACE_BF16 || a.src_mode != kSrcPairList)) return hipErrorInvalidValue;
  const int rb = rank_blocks(r_max);
  if (dtype == ACE_BF16) {
    if (rb == 2) return launch_contract_bf16<2>(a, P, stream);
    if (rb == 4) return launch_contract_bf16<4>(a, P, stream);
    if (rb == 8) return launch_contract_bf16<8>(a, P, stream);
    return launch_contract_bf16<16>(a, P, stream);
  }
  if (rb == 2) return launch_contract_f32<2>(a, P, stream);
  if (rb == 4) return launch_contract_f32<4>(a, P, stream);
  if (rb == 8) return launch_contract_f32<8>(a, P, stream);
  return launch_contract_f32<16>(a, P, stream);
}

}  // namespace ace
