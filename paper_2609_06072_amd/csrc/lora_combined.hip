// Pre-combined adapter input (ACE_INPUT_COMBINED): the down projection of an
// MoE layer whose output is combined over the routed experts with the
// routing weights (Sec. 3.1).  Because that combine is linear, the adapter
// part of the combined output of token t is
//   out[t] += sum_{u: rows of t} s_q B_q A_q z_u,   z_u = sum_{p in u} w_p x_p
// -- one input combination and one adapter evaluation per (token, active
// group) row, the compute-once reuse of Sec. 3.5 carried over to an input
// that differs per routed pair.  Since A_q is linear the launches evaluate
// h_u = s_q A_q z_u as sum_p w_p (s_q A_q x_p):
//
// Forward (h stays in the workspace for the backward: the dense h rows for
// bf16, h_p per pair position for fp32 and for group-keyed rows of single
// pairs, which the combine sums per (token, key)):
//   prep      -- B^T rows [R][d_out] (matrix-core GEMM operand) or B
//                re-strided to [d_out][R] (register GEMM); zero the dense
//                per-token h rows.
//   contract  -- h_p = s_q A_q x_p for every routed pair, in pair order; bf16:
//                its epilogue sums h_u = sum_{p in u} w_p h_p in fp32 and stores
//                the dense rows Hd[t][roff_q..] (a launch of its own over the
//                stored h_p cost 15.6 us beside the contraction's 36 at the
//                Qwen-like shape).
//   combine   -- fp32: h_u from the stored h_p into the dense rows.
//   GEMM      -- out[t] += Hd[t] B^T over K = R (inactive groups hold zeros).
// Backward, with G_t = dOut[t] (every row of token t sees the same gradient):
//   dB_q = sum_u G_t h_u^T                (rows of q)
//   dH_u = s_q B_q^T G_t
//   dA_q = sum_p (w_p dH_{u(p)}) x_p^T    (pairs of q)
//   dx_p += w_p A_q^T dH_{u(p)}
// Launches: prep (A^T, B^T) -> h_u transposed per key (bf16: gathered from the
// forward's dense rows, or the contraction with its row sums; fp32: [contract
// h_p unless the forward's is passed] -> combine) -> contract dH per row (stored per row
// and, times each pair's weight, per pair position) -> expand dx over the
// slots of every row -> weight gradients (dB over rows, dA over pairs).
#include "ace_device.hpp"
#include "ace_internal.hpp"

namespace ace {

namespace {

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

struct FwdLayout {
  size_t hp, Hd, Bm, total;
};

// hp [P][rpad] first, dense h rows [T][R] (a backward reads one or the other,
// see dense_h; the place of hp does not depend on which), the B operand of the
// GEMM ([R][d_out] or [d_out][R]); R <= n_keys * r_max.
FwdLayout fwd_layout(int T, int k, int d_out, int n_keys, int r_max, size_t es) {
  const size_t P = (size_t)T * k;
  const size_t Rb = (size_t)n_keys * r_max;
  FwdLayout w{};
  size_t o = 0;
  w.hp = o;  o += align256(es * P * rank_pad(ACE_F32, r_max));
  w.Hd = o;  o += align256(es * (size_t)T * Rb);
  w.Bm = o;  o += align256(es * Rb * d_out);
  w.total = o;
  return w;
}

struct BwdLayout {
  size_t At, Bt, hp, Ht, dHw, dHrow, part, total;
};

// At [d_in][R], Bt [R][d_out], hp [P][rpad], Ht / dHw [R][ldh], dH rows
// [P][rpad], weight-gradient partials; 256 bytes of slack (the gradient pass
// reads whole 16-byte fragments of Ht / dHw rows past a segment's end).
BwdLayout bwd_layout(int T, int k, int d_in, int d_out, int n_keys, int r_max, size_t es) {
  const size_t P = (size_t)T * k;
  const size_t Rb = (size_t)n_keys * r_max;
  const size_t ldh = (P + 7) & ~(size_t)7;
  const size_t rpad = rank_pad(ACE_F32, r_max);
  BwdLayout w{};
  size_t o = 0;
  w.At = o;    o += align256(es * d_in * Rb);
  w.Bt = o;    o += align256(es * Rb * d_out);
  w.hp = o;    o += align256(es * P * rpad);
  w.Ht = o;    o += align256(es * Rb * ldh);
  w.dHw = o;   o += align256(es * Rb * ldh);
  w.dHrow = o; o += align256(es * P * rpad);
  w.part = o;  o += align256(grads_part_bytes(T, k, d_in, d_out, n_keys, r_max));
  w.total = o + 256;
  return w;
}

// Bd[n][roff_q + r] = B_q[n][r]: B as one [d_out][R] matrix, the layout the
// register GEMM reads its second operand in.
template <typename T>
__global__ __launch_bounds__(kThreads) void restride_b_kernel(const T* B, T* Bd, int d_out,
                                                              KeyTable keys) {
  const int R = keys.R;
  const long i = (long)blockIdx.x * kThreads + threadIdx.x;
  if (i >= (long)d_out * R) return;
  const int n = (int)(i / R), K = (int)(i % R);
  const int q = upper_index(keys.roff, keys.n_keys, K);
  const int r_q = keys.rank[q], roff = keys.roff[q];
  Bd[i] = B[(size_t)d_out * roff + (size_t)n * r_q + (K - roff)];
}

// Ht[roff_q + r][u - offsets[q]] = Hd[t_u][roff_q + r]: the rows' h from the
// forward's dense per-token rows.  A block takes 64 rows; lane l of wave w
// handles row 64 b + l and the rank chunks w, w + 4, ... (eight ranks each),
// so a wave's stores cover 64 consecutive columns.
__global__ __launch_bounds__(kThreads) void gather_h_kernel(const __bf16* Hd, const int32_t* offsets,
                                                            const int32_t* row_token, __bf16* Ht,
                                                            long ldh, KeyTable keys) {
  __shared__ int seg[kMaxKeys + 1];
  for (int i = threadIdx.x; i <= keys.n_keys; i += kThreads) seg[i] = offsets[i];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int u = blockIdx.x * 64 + lane;
  if (u >= seg[keys.n_keys]) return;
  const int q = upper_index(seg, keys.n_keys, u);
  const int r_q = keys.rank[q], roff = keys.roff[q];
  const __bf16* src = Hd + (size_t)row_token[u] * keys.R + roff;
  const long col = u - seg[q];
  const bool vec = ((roff | keys.R | r_q) & 7) == 0;
  for (int r0 = 8 * wave; r0 < r_q; r0 += 32) {
    const bf16x8 v = load_frag<__bf16>(src + r0, r_q - r0, vec);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (r0 + e < r_q) Ht[(size_t)(roff + r0 + e) * ldh + col] = v[e];
  }
}

// h_p = s_q A_q x_p for every routed pair, row-major per pair position.
ContractArgs pair_h_args(const Problem& p, void* hp, int rpad) {
  ContractArgs c{};
  c.src = p.x;
  c.W = p.A;
  c.ldw = p.d_in;
  c.K = p.d_in;
  c.src_mode = kSrcPairList;
  c.k = p.k;
  c.alpha = p.alpha;
  c.plist = p.rt->pair_list;
  c.ppos = p.rt->row_pair;
  c.offsets = p.rt->offsets;
  c.row_token = p.rt->row_token;
  c.row_slots = p.rt->row_slots;
  c.out_row = hp;
  c.rpad = rpad;
  c.keys = p.keys;
  return c;
}

// Where the forward leaves h for the backward: in the dense per-token rows
// (bf16), or as h_p per pair position: fp32, and rows that are single pairs
// (group-keyed), which may share a token and a key, so that their h can't be
// read back from one dense row.  Type and row mode alone decide it.
bool dense_h(const Problem& p) { return p.dtype == ACE_BF16 && p.rt->mode != ACE_ROWS_GROUP_PAIRS; }

// Whether the contraction sums h per row itself (it finds a tile's rows
// through pair_row, which a routing built by hand may leave out: then h_p and
// the combine, as for fp32).
bool sums_rows(const Problem& p) { return dense_h(p) && p.rt->pair_row; }

// bf16: the same, summed per row with the pair weights (h_u), into dense
// per-token rows Hd and/or per key into Ht (either may be null).
hipError_t launch_row_h(const Problem& p, void* Hd, void* Ht, long ldh, int rpad, hipStream_t stream) {
  ContractArgs c = pair_h_args(p, nullptr, rpad);
  c.row_sum = 1;
  c.pair_row = p.rt->pair_row;
  c.pair_w = p.pair_w;
  c.out_dense = Hd;
  c.kslots = 1;
  c.out_t = Ht;
  c.ldh = ldh;
  return launch_contract(p.dtype, c, p.r_max, (long)p.T * p.k, stream);
}

}  // namespace

size_t fwd_combined_ws_bytes(int T, int k, int d_out, int n_keys, int r_max) {
  return fwd_layout(T, k, d_out, n_keys, r_max, sizeof(float)).total;
}

size_t bwd_combined_ws_bytes(int T, int k, int d_in, int d_out, int n_keys, int r_max) {
  return bwd_layout(T, k, d_in, d_out, n_keys, r_max, sizeof(float)).total;
}

hipError_t launch_fwd_combined(const Problem& p, void* y, void* ws, hipStream_t stream) {
  const long P = (long)p.T * p.k;
  const int R = p.keys.R;
  const size_t es = p.dtype == ACE_BF16 ? 2 : 4;
  const int rpad = rank_pad(p.dtype, p.r_max);
  const FwdLayout L = fwd_layout(p.T, p.k, p.d_out, p.keys.n_keys, p.r_max, es);
  char* base = static_cast<char*>(ws);
  // the bf16 GEMM with LDS staging reads B^T rows [R][d_out]; the register
  // GEMM reads [d_out][R]
  const bool rows_op = p.dtype == ACE_BF16 && R % 8 == 0;
  hipError_t e = launch_prep(p, nullptr, rows_op ? base + L.Bm : nullptr, base + L.Hd,
                             (long)p.T * R * (long)es, stream);
  if (e != hipSuccess) return e;
  if (!rows_op) {
    const long n = (long)p.d_out * R;
    const int blocks = (int)((n + kThreads - 1) / kThreads);
    if (p.dtype == ACE_BF16)
      restride_b_kernel<__bf16><<<blocks, kThreads, 0, stream>>>(
          static_cast<const __bf16*>(p.B), reinterpret_cast<__bf16*>(base + L.Bm), p.d_out, p.keys);
    else
      restride_b_kernel<float><<<blocks, kThreads, 0, stream>>>(
          static_cast<const float*>(p.B), reinterpret_cast<float*>(base + L.Bm), p.d_out, p.keys);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (sums_rows(p)) {
    e = launch_row_h(p, base + L.Hd, nullptr, 0, rpad, stream);
  } else {
    e = launch_contract(p.dtype, pair_h_args(p, base + L.hp, rpad), p.r_max, P, stream);
    if (e != hipSuccess) return e;
    e = launch_combine(p, base + L.hp, rpad, nullptr, 0, base + L.Hd, stream);
  }
  if (e != hipSuccess) return e;
  DxArgs d{};
  d.dHf = base + L.Hd;
  d.At = base + L.Bm;
  d.A = base + L.Bm;
  d.dx = y;
  d.T = p.T;
  d.d_in = p.d_out;
  d.R = R;
  d.KR = R;
  return launch_dx_gemm(p.dtype, d, stream);
}

hipError_t launch_bwd_combined(const Problem& p, const void* dy, void* dx, float* dA, float* dB,
                               void* ws, hipStream_t stream) {
  const long P = (long)p.T * p.k;
  const size_t es = p.dtype == ACE_BF16 ? 2 : 4;
  const int rpad = rank_pad(p.dtype, p.r_max);
  const BwdLayout L = bwd_layout(p.T, p.k, p.d_in, p.d_out, p.keys.n_keys, p.r_max, es);
  char* base = static_cast<char*>(ws);
  const long ldh = (long)((((size_t)P) + 7) & ~(size_t)7);
  hipError_t e = launch_prep(p, base + L.At, base + L.Bt, nullptr, 0, stream);
  if (e != hipSuccess) return e;
  if (p.h_fwd && dense_h(p)) {   // the dense rows in the forward's workspace
    const FwdLayout F = fwd_layout(p.T, p.k, p.d_out, p.keys.n_keys, p.r_max, es);
    if (P > 0) {
      gather_h_kernel<<<(int)((P + 63) / 64), kThreads, 0, stream>>>(
          reinterpret_cast<const __bf16*>(static_cast<const char*>(p.h_fwd) + F.Hd), p.rt->offsets,
          p.rt->row_token, reinterpret_cast<__bf16*>(base + L.Ht), ldh, p.keys);
      e = hipGetLastError();
    }
  } else if (sums_rows(p)) {
    e = launch_row_h(p, nullptr, base + L.Ht, ldh, rpad, stream);
  } else {
    // h per pair position: the forward's (its workspace starts with it) or recomputed
    const void* hp = p.h_fwd;
    if (!hp) {
      hp = base + L.hp;
      e = launch_contract(p.dtype, pair_h_args(p, base + L.hp, rpad), p.r_max, P, stream);
      if (e != hipSuccess) return e;
    }
    e = launch_combine(p, hp, rpad, base + L.Ht, ldh, nullptr, stream);
  }
  if (e != hipSuccess) return e;
  // dH_u = s B^T dOut[t_u], per row (for dx) and times w_p per pair position (for dA)
  ContractArgs c{};
  c.src = dy;
  c.W = base + L.Bt;
  c.ldw = p.d_out;
  c.K = p.d_out;
  c.src_mode = kSrcShared;
  c.k = p.k;
  c.alpha = p.alpha;
  c.pair_w = p.pair_w;
  c.offsets = p.rt->offsets;
  c.row_token = p.rt->row_token;
  c.row_slots = p.rt->row_slots;
  c.multi_slot = p.rt->mode == ACE_ROWS_GROUP_DEDUP;
  c.out_row = base + L.dHrow;
  c.rpad = rpad;
  c.out_t = base + L.dHw;
  c.ldh = ldh;
  c.out_t_pairs = 1;
  c.ppos = p.rt->row_pair;
  c.keys = p.keys;
  e = launch_contract(p.dtype, c, p.r_max, P, stream);
  if (e != hipSuccess) return e;
  // dx_p += w_p A_q^T dH_u for every slot of row u
  ExpandArgs x{};
  x.H = base + L.dHrow;
  x.rpad = rpad;
  x.W = base + L.At;
  x.w_key_mul = 1;
  x.w_stride_is_rank = 0;
  x.offsets = p.rt->offsets;
  x.row_token = p.rt->row_token;
  x.row_slots = p.rt->row_slots;
  x.k = p.k;
  x.n_out = p.d_in;
  x.out = dx;
  x.pair_w = p.pair_w;
  x.keys = p.keys;
  x.multi_slot = p.rt->mode == ACE_ROWS_GROUP_DEDUP;
  e = launch_expand(p.dtype, x, p.r_max, P, stream);
  if (e != hipSuccess) return e;
  GradArgs gr{};
  gr.x = p.x;
  gr.dy = dy;
  gr.Hw = base + L.Ht;
  gr.dHt = base + L.dHw;
  gr.ldh = ldh;
  gr.dA = dA;
  gr.dB = dB;
  gr.part = base + L.part;
  gr.offsets = p.rt->offsets;
  gr.row_token = p.rt->row_token;
  gr.row_slots = p.rt->row_slots;
  gr.ppos = p.rt->row_pair;
  gr.plist = p.rt->pair_list;
  gr.k = p.k;
  gr.d_in = p.d_in;
  gr.d_out = p.d_out;
  gr.per_pair = 1;
  gr.combined = 1;
  gr.keys = p.keys;
  return launch_grads(p.dtype, gr, p.r_max, P, stream);
}

}  // namespace ace
