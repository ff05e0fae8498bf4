// Adapted expert projection: the frozen expert GEMM of an MoE layer with the
// adapter update added in its epilogue (Sec. 3.1 base projection W_e x plus
// the Sec. 3.4 shared-adapter update, executed as in Sec. 3.5):
//   y[t*k + j] = W_e xin(t, j) + B_q h_u,   e = topk_ids[t, j], q = key of e,
// where h_u = (alpha / r_q) A_q xin is the shrink of the adapter row u that
// serves the pair (one row per (token, active group) for grouped execution,
// one per pair for expert-wise LoRA), computed beforehand by the contract
// kernel.  y is written once: the adapter's read-modify-write of y is gone.
//
// Three kernels, chosen by the average number of rows per expert (see
// launch_moe_gemm): streaming (few rows), medium tiles and (bf16) large
// tiles.  Each cuts the rows of the expert routing (sorted by expert,
// then token) into tiles of one expert's rows; the contraction runs over d_in
// (x rows against W_e rows, both contiguous along it) and over the adapter
// rank (h rows against B_q rows, from registers), into the same fp32
// accumulators.  The weight rows are the first MFMA operand, so a lane's
// accumulator holds four consecutive output columns of one row.
//
// Medium tiles.  One K-block (64 bytes of every row) per stage; x and W_e
// pieces are copied global -> LDS directly (global_load_lds_dwordx4), a row's
// four 16-byte chunks XOR-swizzled (g_swz) so that the fragment reads of 16
// consecutive rows hit distinct banks.  Wave (wy, wx) owns rows 64*wy .. +64
// and columns 128*wx .. +128.
//
// Block order of the medium and large tiles.  Blocks are dealt to the 8 XCDs
// round-robin; block b takes tile (b % 8) * ceil(n_tiles / 8) + b / 8, so each
// XCD walks a contiguous run of tiles (expert-major): an expert's weight
// slices stay in one L2.
#include <type_traits>

#include "ace_device.hpp"
#include "ace_internal.hpp"

namespace ace {

namespace {

constexpr int kGRowBytes = 64;           // bytes of a row per stage (one K-block)

// Tile geometry: WM x WN waves of 64 rows x 128 columns each, NBUF stages of
// (BM + BN) rows x 64 bytes in LDS.
template <int WM_, int WN_, int NBUF_>
struct GCfg {
  static constexpr int WM = WM_, WN = WN_, NBUF = NBUF_;
  static constexpr int NW = WM * WN, THREADS = 64 * NW;
  static constexpr int BM = 64 * WM, BN = 128 * WN;
  static constexpr int XBYTES = BM * kGRowBytes, STAGE = (BM + BN) * kGRowBytes;
  static constexpr int COPIES = (BM + BN) / 16 / NW;   // 16-row copies per wave per stage
  static_assert((BM + BN) / 16 % NW == 0, "copies must split evenly over the waves");
  static_assert(THREADS >= BM, "one thread per tile row fills the row tables");
};
// Medium tiles: 128 rows x 256 columns, four waves, three stages (72 KB
// of LDS, two blocks per CU), so that an expert's last tile wastes little.
using MoeMid = GCfg<2, 2, 3>;
constexpr int kRowGroup = 8;

// Epilogue passes over column slices so that the C tile [BM][BN/NH + pad]
// fits the stage buffers.
template <class C, typename T>
constexpr int epi_passes() {
  int nh = 1;
  while (C::BM * (C::BN / nh + 16 / (int)sizeof(T)) * (int)sizeof(T) > C::NBUF * C::STAGE) nh *= 2;
  return nh;
}

// Chunk position of a row's 16-byte chunk 0.  Rows 64 bytes apart share a
// bank line; the position differs for any two rows among 8 consecutive ones
// with the same parity and among 16 consecutive ones with the same residue
// mod 4, so a fragment read (16 rows, one chunk each) is free of bank
// conflicts whether the LDS serves 8 or 16 lanes of a 16-byte read per cycle.
__device__ inline int g_swz(int row) { return (((row >> 1) ^ (row >> 3)) & 1) | ((row >> 1) & 2); }

// Number of tiles of BM rows over the key segments offsets[0 .. n_keys]
// (wave-level; every lane gets the total).
__device__ inline int count_tiles(const int32_t* offsets, int n_keys, int BM) {
  constexpr int KPL = kMaxKeys / 64;
  const int lane = threadIdx.x & 63;
  int cnt = 0;
  int prev = offsets[min(lane * KPL, n_keys)];
#pragma unroll
  for (int i = 0; i < KPL; ++i) {
    const int nxt = offsets[min(lane * KPL + i + 1, n_keys)];
    cnt += (nxt - prev + BM - 1) / BM;
    prev = nxt;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
  return cnt;
}

template <typename T, class C>
__global__ __launch_bounds__(C::THREADS, 512 / C::THREADS) void moe_gemm_kernel(MoeArgs a) {
  using F = typename Tr<T>::frag;
  constexpr int PER = Tr<T>::PER, KB = Tr<T>::KB;
  constexpr int BM = C::BM, BN = C::BN, NBUF = C::NBUF, STAGE = C::STAGE, COPIES = C::COPIES;
  constexpr int NT = C::THREADS;
  constexpr int NH = epi_passes<C, T>();       // epilogue passes over column slices
  constexpr int HC = BN / NH;                  // columns per pass
  constexpr int CST = HC + 16 / (int)sizeof(T);
  __shared__ __attribute__((aligned(16))) char smem[NBUF * STAGE];
  __shared__ int s_src[BM];    // x row of each tile row (clamped into the segment)
  __shared__ int s_out[BM];    // y row, -1 past the segment
  __shared__ int s_h[BM];      // adapter row, -1 for none

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  const int wy = wave / C::WN, wx = wave % C::WN;

  // ---- which tile
  const int n_mt = count_tiles(a.offsets, a.E, BM);
  const int n_tiles = n_mt * a.nt;
  const int per_xcd = (n_tiles + kXcds - 1) / kXcds;
  const int bi = blockIdx.x / kXcds;
  const int tile = (blockIdx.x % kXcds) * per_xcd + bi;
  if (bi >= per_xcd || tile >= n_tiles) return;
  const int mt = tile / a.nt, n0 = (tile % a.nt) * BN;
  int e, u0, uend;
  locate_tile(a.offsets, a.E, BM, mt, &e, &u0, &uend);

  if (tid < BM) {
    const int u = u0 + tid;
    const int uc = min(u, uend - 1);
    const int tok = a.row_token[uc];
    const int j = __builtin_ctz(a.row_slots[uc] | 0x80000000u) & 31;
    const int p = tok * a.k + j;
    s_src[tid] = a.per_pair ? p : tok;
    s_out[tid] = u < uend ? p : -1;
    s_h[tid] = (u < uend && a.H) ? a.h_row[p] : -1;
  }
  __syncthreads();

  // A wave whose 64 rows all lie past the expert's last row (the tail of its
  // last tile) skips its matrix work; it still takes part in the copies, the
  // LDS reads and the barriers.  Its accumulators stay zero and are never
  // stored.
  const bool active = u0 + 64 * wy < uend;
  const T* X = static_cast<const T*>(a.x);
  const T* Wt = static_cast<const T*>(a.W) + ((size_t)e * a.d_out + n0) * a.d_in;
  const int d_in = a.d_in, d_out = a.d_out;
  const int nst = (d_in + KB - 1) / KB;

  // ---- copy assignment: lane covers row (lane >> 2) of each 16-row copy,
  // chunk position lane & 3 (global chunk (lane & 3) ^ g_swz(row)).  The
  // swizzle only sees bits 1..3 of the row, i.e. of lane >> 2, so one chunk
  // offset serves every copy; rows are 32-bit element offsets from x (fewer
  // than 2^32 elements, see launch_moe_gemm) or from the tile's first W row.
  const int cpos = lane & 3, crl = lane >> 2;
  const int coff = PER * (cpos ^ g_swz(crl));
  uint32_t roff[COPIES];
#pragma unroll
  for (int i = 0; i < COPIES; ++i) {
    const int blk = wave * COPIES + i;        // 16-row copy index over [x rows | W rows]
    const int row = 16 * blk + crl;
    roff[i] = 16 * blk < BM ? (uint32_t)s_src[row] * (uint32_t)d_in
                            : (uint32_t)min(row - BM, d_out - 1 - n0) * (uint32_t)d_in;
  }
  const uint32_t sbase = lds_addr(smem);
  auto issue = [&](int st) {
    const uint32_t buf = sbase + (st % NBUF) * STAGE;
    const uint32_t kk = (uint32_t)min(st * KB + coff, d_in - PER);
#pragma unroll
    for (int i = 0; i < COPIES; ++i) {
      const int blk = wave * COPIES + i;
      const bool xcopy = 16 * blk < BM;
      dma16((xcopy ? X : Wt) + (roff[i] + kk),
            __builtin_amdgcn_readfirstlane(buf + 16 * blk * kGRowBytes));
    }
  };
#pragma unroll
  for (int s = 0; s < NBUF; ++s)
    if (s < nst) issue(s);

  f32x4 acc[8][4];
#pragma unroll
  for (int nb = 0; nb < 8; ++nb)
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // ---- adapter K-blocks: acc[n][m] += sum_rho B_q[n][rho] h_m[rho]
  if (a.H && active) {
    const int q = a.key_of[e];
    const int r_q = a.keys.rank[q];
    const T* Bq = static_cast<const T*>(a.B) + (size_t)d_out * a.keys.roff[q];
    const T* Hm = static_cast<const T*>(a.H);
    const bool bvec = (r_q % PER) == 0;
    for (int kb = 0; kb * KB < r_q; ++kb) {
      const int rho = kb * KB + PER * g;
      F hf[4], bf[8];
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        const int hr = s_h[64 * wy + 16 * mb + c16];
        hf[mb] = hr >= 0 ? Tr<T>::load(Hm + (size_t)hr * a.rpad + rho) : Tr<T>::zero();
      }
#pragma unroll
      for (int nb = 0; nb < 8; ++nb) {
        const int n = min(n0 + 128 * wx + 16 * nb + c16, d_out - 1);
        bf[nb] = load_frag<T>(Bq + (size_t)n * r_q + rho, r_q - rho, bvec);
      }
#pragma unroll
      for (int nb = 0; nb < 8; ++nb)
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) acc[nb][mb] = Tr<T>::mma(bf[nb], hf[mb], acc[nb][mb]);
    }
  }

  // ---- main loop over d_in, fragments double-buffered in registers: the
  // LDS reads of K-block st + 1 are in flight while the matrix cores work on
  // K-block st.
  // fragment rows 64 wy + 16 mb + c16 (x) and 128 wx + 16 nb + c16 (W): the
  // swizzle again depends on c16 only, so a read is a lane base plus an
  // immediate offset
  const int xl = (64 * wy + c16) * kGRowBytes + ((g ^ g_swz(c16)) << 4);
  const int wl = C::XBYTES + (128 * wx + c16) * kGRowBytes + ((g ^ g_swz(c16)) << 4);
  auto read_frags = [&](int st, F (&xf)[4], F (&wf)[8]) {
    const char* S = smem + (st % NBUF) * STAGE;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) xf[mb] = *reinterpret_cast<const F*>(S + xl + mb * 16 * kGRowBytes);
#pragma unroll
    for (int nb = 0; nb < 8; ++nb)
      wf[nb] = *reinterpret_cast<const F*>(S + wl + nb * 16 * kGRowBytes);
  };
  auto mma_all = [&](const F (&xf)[4], const F (&wf)[8]) {
#pragma unroll
    for (int nb = 0; nb < 8; ++nb)
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) acc[nb][mb] = Tr<T>::mma(wf[nb], xf[mb], acc[nb][mb]);
  };
  // The last K-block may reach past d_in: once it has landed, its chunks past
  // d_in (copies of the clamped last chunk) are cleared in LDS, so no fragment
  // read needs a mask; those of x and of W both, since an infinity times zero
  // is no zero.  Called with stage st landed and published (possibly twice for
  // the last stage: clearing again changes nothing).
  auto clear_tail = [&](int st) {
    if (st != nst - 1 || d_in % KB == 0) return;
    const int valid = (d_in - st * KB) / PER;   // chunks of this K-block inside d_in
    char* S = smem + (st % NBUF) * STAGE;
    for (int i = tid; i < (BM + BN) * 4; i += NT) {   // x rows, then W rows (BM is a multiple of 16)
      const int row = i >> 2, pos = i & 3;
      if ((pos ^ g_swz(row)) >= valid) *reinterpret_cast<u32x4*>(S + row * kGRowBytes + pos * 16) = u32x4{0u, 0u, 0u, 0u};
    }
    __syncthreads();
  };
  // Stage st lives in buffer st % NBUF.  Before K-block st + 1 is read, the
  // barrier also tells that every wave holds K-block st in registers, so
  // its buffer takes stage st + NBUF.
  // Every half-step reads the next K-block unconditionally (clamped to the
  // last one: a repeated read of a landed buffer is harmless), so the reads
  // and the matrix work on the previous block share one basic block.
  F xa[4], wa[8], xb[4], wb[8];
  wait_vmcnt_upto<(NBUF - 1) * COPIES>(min(NBUF - 1, nst - 1) * COPIES);
  __syncthreads();
  clear_tail(0);
  read_frags(0, xa, wa);
  auto half = [&](int st, F (&xc)[4], F (&wc)[8], F (&xn)[4], F (&wn)[8]) {
    // K-block st is in (xc, wc); K-block st + 1 lands in (xn, wn)
    wait_vmcnt_upto<(NBUF - 2) * COPIES>(min(NBUF - 2, nst - 2 - st) * COPIES);
    __syncthreads();
    if (st + NBUF < nst) issue(st + NBUF);
    const int sn = min(st + 1, nst - 1);
    clear_tail(sn);
    read_frags(sn, xn, wn);
    if (active) mma_all(xc, wc);
  };
  for (int st = 0; st < nst; st += 2) {
    half(st, xa, wa, xb, wb);
    if (st + 1 >= nst) break;
    half(st + 1, xb, wb, xa, wa);
  }

  // ---- epilogue: C tile -> LDS [m][n] (over the stage buffers), then whole
  // 16-byte row pieces of y
  T* Cs = reinterpret_cast<T*>(smem);
  T* Y = static_cast<T*>(a.y);
  constexpr int CPR = HC / PER;                 // 16-byte pieces per row and pass
  constexpr int NP = BM * CPR / NT;
  static_assert(BM * CPR % NT == 0, "epilogue pieces must split evenly");
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < 8; ++nb) {
      const int nl = 128 * wx + 16 * nb + 4 * g - h * HC;   // column inside this pass
      if (nl >= 0 && nl < HC) {
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
          T* cp = Cs + (64 * wy + 16 * mb + c16) * CST + nl;
#pragma unroll
          for (int v = 0; v < 4; ++v) cp[v] = (T)acc[nb][mb][v];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int it = tid + i * NT;
      const int m = it / CPR, pc = (it % CPR) * PER;
      const int orow = s_out[m];
      const int col = n0 + h * HC + pc;
      if (orow >= 0 && col < d_out)
        Tr<T>::store(Y + (size_t)orow * d_out + col, *reinterpret_cast<const F*>(Cs + m * CST + pc));
    }
  }
}

// ---------------------------------------------------------------- bf16, large tiles
//
// 256 rows x 256 columns per block, four waves of 128 x 128 (one per SIMD).
//
// What bounds it: the copies' latency.  The L1 returns its lines in order, so
// an x line that hits the L2 waits behind W lines coming from HBM; with one
// 64 KB stage in flight per CU the copies took 1.8 us per stage of 1.0 us of
// matrix work.  So the LDS (all 160 KB) is a ring of five 32 KB slots, each
// freed after half a stage: a half-step works on one half of a wave's rows
// over all 64 contraction indices of the stage (64 matrix instructions),
// while it reads the next half's x fragments and half of the next stage's W
// fragments into registers.  Four slots (128 KB) are then in flight, and
// pieces stay whole cache lines (128 bytes of a row: halves split by
// contraction index would fetch each line of the L2 twice).
//
// Slot P[v] holds what half-step v reads: x unit v + 1 and W unit v + 2, where
// unit u is the half h = u & 1 (64 of each wave's 128 rows) of stage u >> 1.
// The fragment reads and copies are placed between the matrix instructions by
// hand (groups of four): the one wave of a SIMD has nobody to hide behind.
struct Large {
  static constexpr int BM = 256, BN = 256, THREADS = 256;
  static constexpr int KC = 64, ROWB = 2 * KC;            // indices and bytes of a row per stage
  static constexpr int UNIT = 128 * ROWB, SLOT = 2 * UNIT, SLOTS = 5;
  static constexpr int COPIES = 8;                        // 8-row copies per wave and slot
  static constexpr int HC = BN / 2, CST = HC + 8;         // epilogue: column halves
};

// Chunk position of a row's 16-byte chunk 0 (eight chunks per row).  Any 8
// consecutive rows, and any 8 even or odd rows among 16, take 8 positions.
__device__ inline int l_swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// Key of a tile when key q owns ceil(rows / BM) * per tiles, key-major: its
// segment [lo, hi) and the tile's index among the key's tiles (wave-level,
// every lane gets the result; false past the last tile).
__device__ inline bool locate_key(const int32_t* offsets, int n_keys, int BM, int per, int tile,
                                  int* q_out, int* lo_out, int* hi_out, int* rem_out) {
  constexpr int KPL = kMaxKeys / 64;
  const int lane = threadIdx.x & 63;
  int off[KPL + 1], cnt = 0;
#pragma unroll
  for (int i = 0; i <= KPL; ++i) off[i] = offsets[min(lane * KPL + i, n_keys)];
#pragma unroll
  for (int i = 0; i < KPL; ++i) cnt += (off[i + 1] - off[i] + BM - 1) / BM * per;
  int incl = cnt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  const int excl = incl - cnt;
  const unsigned long long hit = __ballot(tile >= excl && tile < incl);
  if (hit == 0ull) return false;
  const int owner = __builtin_ctzll(hit);
  int t = tile - excl, q = 0, lo = 0, hi = 0, rem = 0;
  bool found = false;
#pragma unroll
  for (int i = 0; i < KPL; ++i) {
    const int n = (off[i + 1] - off[i] + BM - 1) / BM * per;
    if (!found && t < n) {
      q = lane * KPL + i;
      lo = off[i];
      hi = off[i + 1];
      rem = t;
      found = true;
    }
    if (!found) t -= n;
  }
  *q_out = __builtin_amdgcn_readfirstlane(__shfl(q, owner, 64));
  *lo_out = __builtin_amdgcn_readfirstlane(__shfl(lo, owner, 64));
  *hi_out = __builtin_amdgcn_readfirstlane(__shfl(hi, owner, 64));
  *rem_out = __builtin_amdgcn_readfirstlane(__shfl(rem, owner, 64));
  return true;
}

// RAGGED: d_in is no multiple of two stages; the chunks past it are zeroed in
// the fragments, behind a branch: done in every half-step, on the one wave of
// a SIMD that has nothing to hide it behind, it cost a sixth (1000 x 2056, 16
// experts, 1000 and 2000 rows each: 141 -> 120 and 228 -> 196 us).  (A second
// loop for the last stages made the compiler spill accumulators.)
// WIDE: x of 4 GiB or more (below 64 GiB): the copies' 32-bit offsets count
// 16-byte chunks instead of bytes (300,000 rows of 8192 through 8 experts of
// 1024 columns: 5.27 ms; the medium tiles 6.57).
template <bool RAGGED, bool WIDE>
__global__ __launch_bounds__(Large::THREADS, 1) void moe_gemm_large_kernel(MoeArgs a) {
  using C = Large;
  using F = bf16x8;
  constexpr int ROWB = C::ROWB, NC = C::COPIES;
  constexpr int OU = WIDE ? 16 : 1;   // bytes per unit of the copies' offsets
  __shared__ __attribute__((aligned(16))) char smem[C::SLOTS * C::SLOT];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  const int wy = wave >> 1, wx = wave & 1;

  // ---- which tile: runs of tiles per XCD; within an expert, groups of up to
  // eight row tiles walk the columns together (their x rows and each
  // column's W rows stay in the XCD's L2)
  const int n_tiles = count_tiles(a.offsets, a.E, C::BM) * a.nt;
  const int per_xcd = (n_tiles + kXcds - 1) / kXcds;
  const int bi = blockIdx.x / kXcds;
  const int tile = (blockIdx.x % kXcds) * per_xcd + bi;
  if (bi >= per_xcd || tile >= n_tiles) return;
  int e, lo, hi, rem;
  if (!locate_key(a.offsets, a.E, C::BM, a.nt, tile, &e, &lo, &hi, &rem)) return;
  const int m_e = (hi - lo + C::BM - 1) / C::BM;
  const int grp = rem / (kRowGroup * a.nt), gsz = min(kRowGroup, m_e - grp * kRowGroup);
  const int ing = rem - grp * kRowGroup * a.nt;
  const int n0 = (ing / gsz) * C::BN;
  const int u0 = lo + (grp * kRowGroup + ing % gsz) * C::BM;

  const __bf16* X = static_cast<const __bf16*>(a.x);
  const __bf16* Wt = static_cast<const __bf16*>(a.W) + (size_t)e * a.d_out * a.d_in;
  const int d_in = a.d_in, d_out = a.d_out;
  const int nst = (d_in + C::KC - 1) / C::KC;

  // pair of a tile row (rows past the segment repeat its last row)
  auto pair_of = [&](int u) {
    const int uc = min(u, hi - 1);
    return a.row_token[uc] * a.k + (__builtin_ctz(a.row_slots[uc] | 0x80000000u) & 31);
  };
  // ---- the adapter's first two K-blocks (h rows of the pairs, B_q rows) into
  // registers ahead of the copies: loads return in order, so behind them each
  // step of the chain pair -> h row -> h would wait for copies from HBM
  F x0[4], x1a[4], x1b[4], wa[16], wb[16];   // x: K-block 0 and 1 of a half, W: [nb + 8 kh]
  const int q = a.H ? a.key_of[e] : 0;
  const int r_q = a.H ? a.keys.rank[q] : 0;
  const __bf16* Bq = static_cast<const __bf16*>(a.B) + (a.H ? (size_t)d_out * a.keys.roff[q] : 0);
  const __bf16* Hm = static_cast<const __bf16*>(a.H);
  const bool bvec = (r_q & 7) == 0;
  int hrow[8];
  if (r_q > 0) {
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
      const int u = u0 + 128 * wy + 16 * mb + c16;
      const int hr = a.h_row[pair_of(u)];   // (rows past the segment: its last row's)
      hrow[mb] = u < hi ? hr : -1;
    }
  }
  auto adapter_load = [&](int kb, F (&f)[16]) {   // B rows, then h rows
    const int rho = kb * 32 + 8 * g;
#pragma unroll
    for (int nb = 0; nb < 8; ++nb) {
      const int n = min(n0 + 128 * wx + 16 * nb + c16, d_out - 1);
      f[nb] = load_frag<__bf16>(Bq + (size_t)n * r_q + rho, r_q - rho, bvec);
    }
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
      f[8 + mb] = hrow[mb] >= 0 ? Tr<__bf16>::load(Hm + (size_t)hrow[mb] * a.rpad + rho) : Tr<__bf16>::zero();
  };

  // ---- copies: waves 0 and 1 copy the x rows of waves (wy = 0, 1), waves 2
  // and 3 the W rows of (wx = 0, 1): of a slot the eight 8-row copies of their
  // 64 rows, lane l the chunk at position l & 7 of row l >> 3.  Rows are
  // offsets (OU) from x or from the tile's first W row; chunks past d_in repeat the
  // row's last one (masked in the fragments of a ragged d_in).
  const int crl = lane >> 3, cpos = lane & 7;
  const bool xwave = wave < 2;
  const char* base = xwave ? reinterpret_cast<const char*>(X)
                           : reinterpret_cast<const char*>(Wt + (size_t)n0 * d_in);
  uint32_t roff[2][NC];   // slots P[v] of even and of odd v
#pragma unroll
  for (int par = 0; par < 2; ++par)
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int h = xwave ? 1 - par : par;   // x unit v + 1, W unit v + 2
      const int row = 128 * (wave & 1) + 64 * h + 8 * i + crl;
      int src;
      if (xwave) {
        const int uc = min(u0 + row, hi - 1);
        src = a.per_pair ? pair_of(uc) : a.row_token[uc];
      } else {
        src = min(row, d_out - 1 - n0);
      }
      roff[par][i] = (uint32_t)src * (uint32_t)(2 * d_in / OU);
    }
  // chunk of the copied row: the swizzle's bit 3 alternates with i
  const int col[2] = {8 * (cpos ^ l_swz(crl)), 8 * (cpos ^ l_swz(8 + crl))};
  const uint32_t cbase = lds_addr(smem) + (xwave ? 0 : C::UNIT) + (wave & 1) * (C::UNIT / 2);
  uint32_t cslot = cbase;             // where this wave's copies of the next slot go
  uint32_t colb[2];                   // column (OU) of a lane's chunk, by copy parity
  auto begin_copies = [&](int v) {    // of slot P[v]
    const int st = max(0, min((v + (xwave ? 1 : 2)) >> 1, nst - 1));
#pragma unroll
    for (int c = 0; c < 2; ++c) colb[c] = 2 * min(st * C::KC + col[c], d_in - 8) / OU;
  };
  auto copy = [&](int par, int i) {
    const char* p = base + (size_t)(roff[par][i] + colb[i & 1]) * OU;
    dma16(p, __builtin_amdgcn_readfirstlane(cslot + i * 1024));
  };
  auto end_copies = [&]() {
    cslot += C::SLOT;
    if (cslot >= cbase + C::SLOTS * C::SLOT) cslot = cbase;
  };
  if (r_q > 0) adapter_load(0, wa);
  if (r_q > 32) adapter_load(1, wb);
#pragma unroll
  for (int v = -2; v < 2; ++v) {
    begin_copies(v);
#pragma unroll
    for (int i = 0; i < NC; ++i) copy(v & 1, i);
    end_copies();
  }

  f32x4 acc[8][8];
#pragma unroll
  for (int nb = 0; nb < 8; ++nb)
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  // adapter K-blocks: acc[n][m] += sum_rho B_q[n][rho] h_m[rho]
  auto adapter_mma = [&](const F (&f)[16]) {
#pragma unroll
    for (int nb = 0; nb < 8; ++nb)
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) mfma_acc(acc[nb][mb], f[nb], f[8 + mb]);
  };
  if (r_q > 0) adapter_mma(wa);
  if (r_q > 32) adapter_mma(wb);
  for (int kb = 2; kb * 32 < r_q; ++kb) {
    adapter_load(kb, wa);
    adapter_mma(wa);
  }

  // ---- main loop over d_in.  Fragment rows 64 wy + 16 mb + c16 of an x unit
  // and 64 wx + 16 nb + c16 of a W unit: their swizzle depends on c16 only;
  // K-block kh of the stage is chunk 4 kh + g, the lane's base with bit 6
  // flipped for kh = 1.
  const int xl = (64 * wy + c16) * ROWB + ((g ^ l_swz(c16)) << 4);
  const int wl = C::UNIT + (64 * wx + c16) * ROWB + ((g ^ l_swz(c16)) << 4);
  int rslot = 0;                      // slot that the half-step reads
  // Half-step v = 2 st + h (h = PAR): matrix work on (xc, wc) for the wave's
  // row blocks 4 h .. 4 h + 3; reads slot P[v]: the next half's x fragments
  // into xn, the W fragments nb = 4 h .. 4 h + 3 of stage st + 1 into wn;
  // copies slot P[v + 4] over the one that half-step v - 1 read.
  auto half = [&](auto par_c, auto mma_c, int v, F (&x1)[4], F (&wc)[16],
                  F (&x1n)[4], F (&wn)[16]) {
    constexpr int PAR = decltype(par_c)::value;
    constexpr bool MMA = decltype(mma_c)::value;
    // this wave's reads of P[v - 1] are done and its copies of P[v] have
    // landed (three later slots may be in flight); after the barrier that
    // holds for every wave
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x4078);   // vmcnt(24) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    const char* xs = smem + rslot + xl;
    const char* ws = smem + rslot + wl;
    const char* xs1 = smem + rslot + (xl ^ 64);
    const char* ws1 = smem + rslot + (wl ^ 64);
    begin_copies(v + 4);
    const int c = (v >> 1) * C::KC + 8 * g;
    const bool past = RAGGED && MMA && (v >> 1) * C::KC + C::KC > d_in;   // wave-uniform
    if (PAR == 0 && past) {
#pragma unroll
      for (int nb = 0; nb < 8; ++nb) {
        if (c >= d_in) wc[nb] = Tr<__bf16>::zero();
        if (c + 32 >= d_in) wc[nb + 8] = Tr<__bf16>::zero();
      }
    }
    if (past) {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        if (c >= d_in) x0[mb] = Tr<__bf16>::zero();
        if (c + 32 >= d_in) x1[mb] = Tr<__bf16>::zero();
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i < 8) {   // groups 0..7 work on K-block 0, groups 8..15 on K-block 1
        if (i < 4) x1n[i] = *reinterpret_cast<const F*>(xs1 + i * 16 * ROWB);
        wn[4 * PAR + (i & 3) + 8 * (i >> 2)] =
            *reinterpret_cast<const F*>((i < 4 ? ws : ws1) + (i & 3) * 16 * ROWB);
        copy(PAR, i);
      }
      if (i >= 8 && i < 12) x0[i - 8] = *reinterpret_cast<const F*>(xs + (i - 8) * 16 * ROWB);
      if constexpr (MMA) {
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
          const int nb = i & 7, kh = i >> 3;
          mfma_acc(acc[nb][4 * PAR + mb], wc[nb + 8 * kh], kh ? x1[mb] : x0[mb]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    end_copies();
    rslot = rslot == (C::SLOTS - 1) * C::SLOT ? 0 : rslot + C::SLOT;
  };
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  using Yes = std::true_type;
  using No = std::false_type;
  half(P0{}, No{}, -2, x1a, wb, x1b, wa);
  half(P1{}, No{}, -1, x1b, wb, x1a, wa);
  for (int st = 0; st < nst; st += 2) {   // two stages: the W fragments change registers
    half(P0{}, Yes{}, 2 * st, x1a, wa, x1b, wb);
    half(P1{}, Yes{}, 2 * st + 1, x1b, wa, x1a, wb);
    half(P0{}, Yes{}, 2 * st + 2, x1a, wb, x1b, wa);
    half(P1{}, Yes{}, 2 * st + 3, x1b, wb, x1a, wa);
  }
  wait_vmcnt<0>();   // copies past the last stage (repeats of it)
  mfma_done();
  __builtin_amdgcn_sched_barrier(0);

  // ---- epilogue: column halves of the tile through LDS, whole 16-byte pieces of y rows
  __bf16* Cs = reinterpret_cast<__bf16*>(smem);
  int* s_out = reinterpret_cast<int*>(smem + C::BM * C::CST * 2);   // y row of each tile row, -1 past the segment
  __bf16* Y = static_cast<__bf16*>(a.y);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    __syncthreads();
    if (h == 0) s_out[tid] = u0 + tid < hi ? pair_of(u0 + tid) : -1;
    if (wx == h) {
#pragma unroll
      for (int nb = 0; nb < 8; ++nb)
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) {
          const f32x4 v = acc[nb][mb];
          const bf16x4 o = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
          *reinterpret_cast<bf16x4*>(Cs + (128 * wy + 16 * mb + c16) * C::CST + 16 * nb + 4 * g) = o;
        }
    }
    __syncthreads();
    constexpr int CPR = C::HC / 8;
#pragma unroll 4
    for (int it = tid; it < C::BM * CPR; it += C::THREADS) {
      const int m = it / CPR, pc = (it % CPR) * 8;
      const int orow = s_out[m], cc = n0 + h * C::HC + pc;
      if (orow >= 0 && cc < d_out)
        Tr<__bf16>::store(Y + (size_t)orow * d_out + cc, *reinterpret_cast<const F*>(Cs + m * C::CST + pc));
    }
  }
}

// ---------------------------------------------------------------- few rows per expert
//
// Decode batches: every active expert's weights are read for a handful of
// rows, so HBM bounds the call and a block streams W.  It takes up to 16 NRB
// rows of one expert and 64 columns; wave w owns 16 columns over the whole
// contraction.  Stages of 256 bytes of the 64 W rows and of the x rows are
// copied global -> LDS, two in LDS (three or four blocks per CU keep 60 to
// 70 KB in flight); W goes through non-temporal, it is read once.
// OLMoE-like, 48 tokens (three projections of 268 MB of weights): 231 -> 200 us
// a pass against the 128-row tiles, W at 5.0 TB/s; without the non-temporal
// policy 217 us.
template <typename T, int NRB>
struct MStream {
  static constexpr int ROWB = 256, KC = ROWB / (int)sizeof(T), NBUF = 2;
  static constexpr int BM = 16 * NRB, BN = 64, NS = 4;     // NS: 4-row W copies per wave and stage
  static constexpr int WBYTES = BN * ROWB, STAGE = WBYTES + BM * ROWB;
};

template <typename T, int NRB>
__global__ __launch_bounds__(256) void moe_stream_kernel(MoeArgs a) {
  using C = MStream<T, NRB>;
  using F = typename Tr<T>::frag;
  constexpr int PER = Tr<T>::PER, KB = Tr<T>::KB, KC = C::KC, ROWB = C::ROWB, NBUF = C::NBUF;
  __shared__ __attribute__((aligned(16))) char smem[NBUF * C::STAGE];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  const int mt = blockIdx.x / a.nt, n0 = (blockIdx.x % a.nt) * C::BN;
  int e, u0, u_end;
  if (!locate_tile(a.offsets, a.E, C::BM, mt, &e, &u0, &u_end)) return;   // block-uniform
  e = __builtin_amdgcn_readfirstlane(e);
  const int d_in = a.d_in, d_out = a.d_out;
  const T* X = static_cast<const T*>(a.x);
  const T* Wt = static_cast<const T*>(a.W) + (size_t)e * d_out * d_in;
  auto pair_of = [&](int u) {   // (rows past the segment: its last row)
    const int uc = min(u, u_end - 1);
    return a.row_token[uc] * a.k + (__builtin_ctz(a.row_slots[uc] | 0x80000000u) & 31);
  };
  // copies: lane l takes the chunk at position l & 15 of row l >> 4 of a
  // 4-row copy; a row's chunk 0 sits at position row & 15
  const int crow = lane >> 4, cpos = lane & 15;
  const T* wsrc[C::NS];
  const T* xsrc[NRB];
  int wcol[C::NS], xcol[NRB];
#pragma unroll
  for (int i = 0; i < C::NS; ++i) {
    const int row = 16 * wave + 4 * i + crow;
    wsrc[i] = Wt + (size_t)min(n0 + row, d_out - 1) * d_in;
    wcol[i] = PER * (cpos ^ (row & 15));
  }
#pragma unroll
  for (int i = 0; i < NRB; ++i) {
    const int row = 4 * (wave * NRB + i) + crow;
    const int p = pair_of(u0 + row);
    xsrc[i] = X + (size_t)(a.per_pair ? p : p / a.k) * d_in;
    xcol[i] = PER * (cpos ^ (row & 15));
  }
  // x copies of this wave that hold rows of the tile
  const int nx = min(NRB, max(0, (u_end - u0 + 3) / 4 - wave * NRB));
  const int nst = (d_in + KC - 1) / KC;
  const uint32_t sbase = lds_addr(smem);
  auto issue = [&](int st) {   // columns past d_in repeat the row's last chunk (masked at the reads)
    const uint32_t buf = sbase + (st % NBUF) * C::STAGE;
    const int k0 = st * KC;
#pragma unroll
    for (int i = 0; i < C::NS; ++i)
      dma16_nt(wsrc[i] + min(k0 + wcol[i], d_in - PER),
               __builtin_amdgcn_readfirstlane(buf + (16 * wave + 4 * i) * ROWB));
#pragma unroll
    for (int i = 0; i < NRB; ++i)
      if (i < nx)
        dma16(xsrc[i] + min(k0 + xcol[i], d_in - PER),
              __builtin_amdgcn_readfirstlane(buf + C::WBYTES + 4 * (wave * NRB + i) * ROWB));
  };
  f32x4 acc[NRB];
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib) acc[ib] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < NBUF - 1; ++p)
    if (p < nst) issue(p);
  auto begin_stage = [&](int st) {
    wait_vmcnt_upto<(NBUF - 2) * (C::NS + NRB)>(min(NBUF - 2, nst - 1 - st) * (C::NS + nx));
    __syncthreads();
    if (st + NBUF - 1 < nst) issue(st + NBUF - 1);
  };
  auto kblock = [&](int st, int kb, bool ragged) {
    const char* S = smem + (st % NBUF) * C::STAGE;
    const int chunk = ((kb * 4 + g) ^ c16) << 4;   // rows 16 i + c16
    F wf = *reinterpret_cast<const F*>(S + (16 * wave + c16) * ROWB + chunk);
    const bool past = ragged && st * KC + kb * KB + PER * g >= d_in;
    if (past) wf = Tr<T>::zero();
#pragma unroll
    for (int ib = 0; ib < NRB; ++ib) {
      F xf = *reinterpret_cast<const F*>(S + C::WBYTES + (16 * ib + c16) * ROWB + chunk);
      if (past) xf = Tr<T>::zero();
      acc[ib] = Tr<T>::mma(wf, xf, acc[ib]);   // D[column][row]
    }
  };
  const int nst_full = d_in / KC;
  for (int st = 0; st < nst_full; ++st) {
    begin_stage(st);
#pragma unroll
    for (int kb = 0; kb < KC / KB; ++kb) kblock(st, kb, false);
  }
  if (nst_full < nst) {
    begin_stage(nst_full);
#pragma unroll
    for (int kb = 0; kb < KC / KB; ++kb)
      if (nst_full * KC + kb * KB < d_in) kblock(nst_full, kb, true);
  }
  // the adapter's K-blocks, then the rows of y
  int orow[NRB];
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib) {
    const int u = u0 + 16 * ib + c16;
    orow[ib] = u < u_end ? pair_of(u) : -1;
  }
  if (a.H) {
    const int q = a.key_of[e];
    const int r_q = a.keys.rank[q];
    const T* Bq = static_cast<const T*>(a.B) + (size_t)d_out * a.keys.roff[q];
    const T* Hm = static_cast<const T*>(a.H);
    const bool bvec = (r_q % PER) == 0;
    const int n = min(n0 + 16 * wave + c16, d_out - 1);
    int hrow[NRB];
#pragma unroll
    for (int ib = 0; ib < NRB; ++ib) hrow[ib] = orow[ib] >= 0 ? a.h_row[orow[ib]] : -1;
    for (int kb = 0; kb * KB < r_q; ++kb) {
      const int rho = kb * KB + PER * g;
      const F bf = load_frag<T>(Bq + (size_t)n * r_q + rho, r_q - rho, bvec);
#pragma unroll
      for (int ib = 0; ib < NRB; ++ib) {
        const F hf = hrow[ib] >= 0 ? Tr<T>::load(Hm + (size_t)hrow[ib] * a.rpad + rho) : Tr<T>::zero();
        acc[ib] = Tr<T>::mma(bf, hf, acc[ib]);
      }
    }
  }
  T* Y = static_cast<T*>(a.y);
  const int col = n0 + 16 * wave + 4 * g;   // four columns, all inside d_out or none
#pragma unroll
  for (int ib = 0; ib < NRB; ++ib)
    if (orow[ib] >= 0 && col < d_out) {
      typedef __attribute__((ext_vector_type(4))) T T4;
      const f32x4 v = acc[ib];
      *reinterpret_cast<T4*>(Y + (size_t)orow[ib] * d_out + col) = T4{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
    }
}

template <typename T, int NRB>
hipError_t launch_moe_stream(MoeArgs a, long P, hipStream_t stream) {
  using C = MStream<T, NRB>;
  a.nt = (a.d_out + C::BN - 1) / C::BN;
  const long grid = ((P + C::BM - 1) / C::BM + a.E) * a.nt;
  if (grid > 0x7fffffffL) return hipErrorInvalidConfiguration;
  if (grid > 0) moe_stream_kernel<T, NRB><<<(int)grid, 256, 0, stream>>>(a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_moe_mid(MoeArgs a, long P, hipStream_t stream) {
  using C = MoeMid;
  a.nt = (a.d_out + C::BN - 1) / C::BN;
  const long max_tiles = ((P + C::BM - 1) / C::BM + a.E) * a.nt;
  const long grid = (max_tiles + kXcds - 1) / kXcds * kXcds;
  if (grid > 0x7fffffffL) return hipErrorInvalidConfiguration;
  if (grid > 0) moe_gemm_kernel<T, C><<<(int)grid, C::THREADS, 0, stream>>>(a);
  return hipGetLastError();
}

hipError_t launch_moe_large(MoeArgs a, long P, bool wide, hipStream_t stream) {
  a.nt = (a.d_out + Large::BN - 1) / Large::BN;
  const long max_tiles = ((P + Large::BM - 1) / Large::BM + a.E) * a.nt;
  const long grid = (max_tiles + kXcds - 1) / kXcds * kXcds;
  if (grid > 0x7fffffffL) return hipErrorInvalidConfiguration;
  const bool ragged = a.d_in % (2 * Large::KC) != 0;
  if (wide && ragged) moe_gemm_large_kernel<true, true><<<(int)grid, Large::THREADS, 0, stream>>>(a);
  else if (wide) moe_gemm_large_kernel<false, true><<<(int)grid, Large::THREADS, 0, stream>>>(a);
  else if (ragged) moe_gemm_large_kernel<true, false><<<(int)grid, Large::THREADS, 0, stream>>>(a);
  else moe_gemm_large_kernel<false, false><<<(int)grid, Large::THREADS, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace

// bf16: which kernel, by the average number of rows per expert, P / E.  A
// second tile of an expert costs its weights a second time, so an average
// close to a tile's rows already loses (random routings, weights out of every
// cache, us a call: streaming with 16 / 32 / 64 rows, medium, large; even
// routing, then one with popularity ~ 1 / rank^0.8):
//   2048 x 1024, 64 experts (256 medium tiles of one per expert)
//      8 rows   54 /  60 /  56,  69,  76      57 /  58 /  57,  71,  76
//     32 rows   86 /  71 /  60,  70,  77      83 /  67 /  67,  95,  84
//     48 rows  111 /  92 /  70,  70,  78     105 /  87 /  75,  93, 121
//     64 rows  134 / 104 /  84,  71,  79     129 /  99 /  81,  96, 119
//    192 rows  277 / 204 / 173,  95,  83     289 / 209 / 177, 101, 118
//    400 rows  524 / 369 / 310, 166, 124     532 / 373 / 311, 163, 124
//   1024 x 2048, 64 experts (512)
//     24 rows   69 /  53 /  60,  56,  75      68 /  60 /  64,  73,  76
//     32 rows   82 /  67 /  62,  57,  76      81 /  66 /  68,  75,  78
//   4096 x 14336, 8 experts (448)
//     16 rows  203 / 182 / 184, 177, 210     199 / 180 / 182, 179, 210
//     32 rows  346 / 237 / 195, 183, 208     325 / 212 / 193, 191, 208
//     64 rows  633 / 389 / 282, 195, 210     632 / 375 / 253, 207, 210
//   14336 x 4096, 8 experts (128)
//     24 rows  270 / 141 / 145, 287, 309     252 / 192 / 145, 293, 307
//     64 rows  558 / 373 / 329, 305, 303     556 / 346 / 275, 316, 307
//   1000 x 2056, 16 experts (144)
//     24 rows   31 /  22 /  24,  34,  36      35 /  24 /  28,  37,  36
//     64 rows   71 /  46 /  34,  38,  37      71 /  46 /  33,  42,  42
// So 32-row tiles end at 20 rows, 64-row tiles at 48; where the medium tiles
// leave CUs idle, at 28 (contractions below 4096) and 64; and where there are
// medium tiles for all CUs one and a half times, they take over from the
// 32-row tiles at 24.
constexpr long kStream16 = 8, kStream32 = 20, kStream64 = 48, kStream32Few = 28, kStream64Few = 64, kMidMany = 24;
constexpr long kLargeRows = 192;

// fp32, whose matrix units bound every tile.  Streaming with 16 / 32 / 64
// rows, medium tiles, us a call: 1024 x 2048, 16 experts:
//    24 rows    37 / 40 / 48, 138            100 rows   113 / 98 / 90, 142
//   160 rows   155 / 131 / 128, 141          250 rows   240 / 197 / 184, 276
//  1200 rows  1060 / 832 / 769, 682         2500 rows  2215 / 1750 / 1548, 1337
// 4096 x 14336, 8 experts:
//   250 rows  4654 / 2819 / 2421, 2657      2500 rows  45811 / 27690 / 22364, 18489
// From 160 rows on the two compare by rounds: a CU takes one medium tile after
// the other (two at once are no faster), so the call takes as long as the
// fullest CU, at 1.2 times the rate per element of y of the streaming kernel,
// whose small blocks even out.  Both count half a tile lost per expert.
// (Balanced routings of about 100 rows fill the medium tiles without that loss:
// 2048 x 1024, 64 experts 288 against 354; uneven ones at the same size 550 and
// 390, which the host can't tell apart.)
constexpr long kStream16F32 = 8, kStream32F32 = 160;

bool mid_f32(const MoeArgs& a, long P) {
  const long cus = device_cu_count(), BM = MoeMid::BM, BN = MoeMid::BN;
  const long tiles = (P / BM + a.E / 2) * ((a.d_out + BN - 1) / BN);
  return 5 * ((tiles + cus - 1) / cus * cus) * BM * BN < 6 * (P + 32 * (long)a.E) * a.d_out;
}

hipError_t launch_moe_gemm(int dtype, const MoeArgs& a, long P, hipStream_t stream) {
  // x rows are 32-bit offsets: elements in the medium tiles, bytes or 16-byte
  // chunks in the large ones; the streaming kernel's are pointers
  const long x_elems = (a.per_pair ? P : P / a.k) * a.d_in;
  const bool mid = x_elems < (1L << 32), large = 2 * x_elems < (1L << 36);
  if (dtype == ACE_F32) {
    if (P <= kStream16F32 * a.E) return launch_moe_stream<float, 1>(a, P, stream);
    if (P <= kStream32F32 * a.E) return launch_moe_stream<float, 2>(a, P, stream);
    if (mid && mid_f32(a, P)) return launch_moe_mid<float>(a, P, stream);
    return launch_moe_stream<float, 4>(a, P, stream);
  }
  const long cus = device_cu_count(), tiles = (long)a.E * ((a.d_out + MoeMid::BN - 1) / MoeMid::BN);
  const bool many = 2 * tiles >= 3 * cus, few = 4 * tiles < 3 * cus;   // medium tiles, one per expert
  const long stream32 = many ? kMidMany : few && a.d_in < 4096 ? kStream32Few : kStream32;
  if (P <= kStream16 * a.E) return launch_moe_stream<__bf16, 1>(a, P, stream);
  if (P <= stream32 * a.E) return launch_moe_stream<__bf16, 2>(a, P, stream);
  if (!many && P <= (few ? kStream64Few : kStream64) * a.E) return launch_moe_stream<__bf16, 4>(a, P, stream);
  if (large && (P >= kLargeRows * a.E || !mid)) return launch_moe_large(a, P, 2 * x_elems >= (1L << 32), stream);
  if (mid) return launch_moe_mid<__bf16>(a, P, stream);
  return launch_moe_stream<__bf16, 4>(a, P, stream);
}

}  // namespace ace
