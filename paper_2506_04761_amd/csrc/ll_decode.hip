// Log-linear Mamba-2 and Gated DeltaNet decoding: one token per call, O(log t) state per head
// (Sec. 3.2).  The Mamba-2 step is described here, the Gated DeltaNet step at k_gdn_decode_step.
//
// Per (b, h) the state is the list of Fenwick level states S^(l) (d_v x d_k).  Token t (0-based)
// updates it as the recurrent form does: for t >= 1, with p = lssb(t), level p+1 receives the
// sum of levels 0..p, levels 1..p are emptied, higher levels carry over, and every carried or
// merged level is multiplied by alpha_t; then level 0 becomes v_t k_t^T.  The output is
// o_t = sum_l lambda_t^(l) S_t^(l) q_t (Eq. 3 read-out).
//
// Storage (one caller-owned buffer, carved by decode_layout):
//   S      [B*H][L][d_v][d_k] fp32   levels LOGW + 1 .. L-1, each kept as c_l * S_stored; the slots
//                                    below them hold the head's window (DecodeWindow)
//   scale  [2][B*H][L]        fp32   c_l, double-buffered by step parity (read t-1, write t)
//   f0     [2][B*H][d_v + d_k] fp32  level 0 in factored form (k_gdn_decode_plain)
//
// Window.  The tokens since the last multiple of W = 2^LOGW are kept as their rows of k and v, not
// as matrices: within one aligned window no level above LOGW changes but for its decay, and the
// levels 0 .. LOGW are sums over the window's own tokens,
//     sum_{s in window, s <= t} lambda_t^(l(t,s)) (alpha_{s+1} .. alpha_t) (k_s . q_t) v_s.
// The step that opens the next window (t % W == 0) merges the full window and the levels
// LOGW + 1 .. p, p = lssb(t), into level p + 1.  So a step reads the nonempty levels above LOGW and
// at most W rows, and writes a matrix once in W steps; kept as matrices, levels 1 .. LOGW cost half
// of LOGW more level reads and one level write at every step.  The decays are applied lazily, through
// one fp32 scale per level and one per window token (double-buffered by step parity like the scales).
// W = 8, 16 or 32 by the batch's size (decode_log_window).  Bound: reading the levels.  1024 heads, d = 128,
// bf16, W = 32, positions 3000 .. 3031: 111 -> 64 us a step, 5 levels (335 MB) at 5.2 TB/s against 8 read and
// one written; 54 us with the levels that have decayed to nothing left out.
//
// Work split: grid (d_v / (16 RB), B*H), 256 threads; thread (row r = tid / 16, part c = tid % 16)
// owns d_v rows 16 (RB blockIdx.x + i) + r, i < RB, and 16-byte pieces c, c + 16, .. of every d_k
// row; row sums are reduced over the 16 lanes of the row.  Workgroups of one head share the window and
// the scales, written only by workgroup x = 0: into slot t % W, which no other workgroup of the launch
// reads, into the other parity, or into the other of the two window buffers.
#include <type_traits>

#include "../../include/libloglinear.h"
#include "ll_device.hpp"

namespace ll {

constexpr int kDecodeThreads = 256;
constexpr int kDecodeMaxLevels = 32;

struct DecodeLayout {
  int64_t S = 0, scale = 0, f0 = 0, total = 0;
};

DecodeLayout decode_layout(int64_t B, int64_t H, int64_t dk, int64_t dv, int64_t L) {
  auto al = [](int64_t x) { return (x + 255) & ~int64_t(255); };
  const int64_t BH = B * H;
  DecodeLayout d;
  int64_t cur = 0;
  d.S = cur; cur += al(BH * L * dv * dk * 4);
  d.scale = cur; cur += al(2 * BH * L * 4);
  d.f0 = cur; cur += al(2 * BH * (dv + dk) * 4);
  d.total = cur;
  return d;
}

// Sum over the 16 (8) lanes of a row, received by every lane (DPP; a row's lanes are active together).
template <int CTRL>
__device__ inline float dpp_add(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
__device__ inline float sum16(float x) {  // rotations by 8, 4, 2, 1
  return dpp_add<0x121>(dpp_add<0x122>(dpp_add<0x124>(dpp_add<0x128>(x))));
}
__device__ inline float sum8(float x) {  // neighbours, pairs, then the mirrored half row
  return dpp_add<0x141>(dpp_add<0x4e>(dpp_add<0xb1>(x)));
}

// A d_k row dealt to LANES lanes in pieces of VEC consecutive entries: lane c holds entries
// LANES VEC j + VEC c .. + VEC - 1 of piece j, so that the lanes of a row read consecutive bytes.
template <int DK, int LANES = 16>
struct RowPart {
  static constexpr int NPT = DK / LANES, VEC = NPT < 4 ? NPT : 4, PIECES = NPT / VEC;
  static_assert(LANES * VEC * PIECES == DK, "whole pieces");
  // ALIGN: of the rows; a caller's q and k may begin at any element
  template <int ALIGN = 0, typename T>
  __device__ static void load(const T* row, int c, float (&x)[NPT]) {
    typedef T vec __attribute__((ext_vector_type(VEC), aligned(ALIGN ? ALIGN : VEC * sizeof(T))));
#pragma unroll
    for (int j = 0; j < PIECES; ++j) {
      const vec y = *reinterpret_cast<const vec*>(row + LANES * VEC * j + VEC * c);
#pragma unroll
      for (int e = 0; e < VEC; ++e) x[VEC * j + e] = to_f32(y[e]);
    }
  }
  template <typename T>
  __device__ static void store(T* row, int c, const float (&x)[NPT]) {
    typedef T vec __attribute__((ext_vector_type(VEC)));
#pragma unroll
    for (int j = 0; j < PIECES; ++j) {
      vec y;
#pragma unroll
      for (int e = 0; e < VEC; ++e) y[e] = from_f32<T>(x[VEC * j + e]);
      *reinterpret_cast<vec*>(row + LANES * VEC * j + VEC * c) = y;
    }
  }
  __device__ static float dot(const float (&x)[NPT], const float (&y)[NPT]) {
    float a = 0.f;
#pragma unroll
    for (int i = 0; i < NPT; ++i) a += x[i] * y[i];
    return a;
  }
};

// Storage of a window's rows: that of k and v, but fp32 for the shape compiled for both types, so that steps of
// either type may follow each other on one state (bf16 values are exact in it).
template <typename T, int DK, int DV>
using WindowRow = std::conditional_t<DK == 64 && DV == 64, float, T>;

// One head's window, in its level slots 0 .. min(LOGW, L - 1) (levels 0 .. LOGW are never stored as
// matrices).  Two buffers alternate by window, so that the step that opens a window can store its
// token while other workgroups still read the full one.  With L - 1 < LOGW levels the state holds
// fewer than W tokens and one buffer of 2^(L-1) slots is used.
template <typename T, int DK, int DV, int LOG>
struct DecodeWindow {
  static constexpr int LOGW = LOG, W = 1 << LOG;
  T *k, *v;              // [cap][d_k], [cap][d_v]
  float *beta, *alpha;   // [cap] (Gated DeltaNet)
  float* gram;           // [cap][cap] k_s . k_r for r < s (Gated DeltaNet)
  static constexpr int buf_bytes(int cap) {
    return (int)((cap * (DK + DV) * sizeof(T) + cap * 8 + cap * cap * 4 + 15) & ~size_t(15));
  }
  static constexpr int dec_bytes(int cap) { return (2 * (cap + 1) * 4 + 15) & ~15; }
  static_assert(dec_bytes(W) + 2 * buf_bytes(W) <= (LOGW + 1) * DK * DV * 4, "the window fits in its levels' slots");
  static_assert(dec_bytes(1) + buf_bytes(1) <= DK * DV * 4 && dec_bytes(2) + buf_bytes(2) <= 2 * DK * DV * 4 &&
                    dec_bytes(W / 2) + buf_bytes(W / 2) <= LOGW * DK * DV * 4,
                "so does a shorter one");
  __device__ static int cap(int L) { return L - 1 >= LOGW ? W : 1 << (L - 1); }
  // decays of the window's tokens up to the step of parity `par`, [cap]; then the whole window's
  __device__ static float* dec(float* head, int L, int64_t par) { return head + (par & 1) * (cap(L) + 1); }
  __device__ DecodeWindow(float* head, int L, int64_t window) {
    const int n = cap(L);
    char* p = reinterpret_cast<char*>(head) + dec_bytes(n) + (window & 1) * buf_bytes(n);
    k = reinterpret_cast<T*>(p);
    v = k + n * DK;
    beta = reinterpret_cast<float*>(v + n * DV);
    alpha = beta + n;
    gram = alpha + n;
  }
};

// The slot of lane c's u-th token in a window of i tokens, -1 past its end.  Slot i is the step's own: workgroup
// x = 0 writes it while the head's other workgroups run, so none of them may read it, nor a later one.
constexpr int window_slot(int c, int u, int i) { return c + 16 * u < i ? c + 16 * u : -1; }
constexpr bool window_slots_ok(int W) {
  for (int i = 0; i < W; ++i) {
    int n = 0;  // every earlier token has one lane
    for (int u = 0; u < (W + 15) / 16; ++u)
      for (int c = 0; c < 16; ++c) {
        if (window_slot(c, u, i) >= i) return false;
        n += window_slot(c, u, i) >= 0;
      }
    if (n != i) return false;
  }
  return true;
}
static_assert(window_slots_ok(8) && window_slots_ok(16) && window_slots_ok(32), "a step reads the tokens before its own, each once");

// The nonempty levels above `l0 - 1` (bit i of `rest`: level l0 + i), lowest first, KB at a time.
template <int KB>
struct LevelBatch {
  int l[KB], n;
  __device__ void next(int64_t& rest, int& l0) {
    n = 0;
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      l[b] = 0;
      if (rest) {
        const int sh = __builtin_ctzll((unsigned long long)rest);
        l[b] = l0 + sh;
        rest >>= sh + 1;
        l0 += sh + 1;
        n = b + 1;
      }
    }
  }
};

template <typename T, int DK, int DV, int LOGW, int RB, bool MERGE>
__global__ __launch_bounds__(kDecodeThreads) void k_decode_step(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, const float* __restrict__ log_alpha,
    const float* __restrict__ lam, T* __restrict__ o, float* __restrict__ S, const float* __restrict__ scale_in,
    float* __restrict__ scale_out, int64_t t, int L) {
  typedef RowPart<DK> RP;
  typedef WindowRow<T, DK, DV> Row;
  typedef DecodeWindow<Row, DK, DV, LOGW> Win;
  constexpr int NPT = RP::NPT, W = Win::W;
  constexpr int KB = RB >= 4 ? 1 : 4;  // levels loaded together
  __shared__ float p_s[W];
  constexpr float kLeftOut = -0.f;  // (x + 0 is never -0)
  const int64_t bh = blockIdx.y;
  const int tid = threadIdx.x, r = tid >> 4, c = tid & 15;
  const int row0 = blockIdx.x * 16 * RB + r;  // rows row0 + 16 x
  const int i = (int)(t & (W - 1));           // the token's slot; the window holds i tokens before it
  float* Sh = S + bh * (int64_t)L * DV * DK;
  const Win win(Sh, L, t >> LOGW);
  const float* dec_in = Win::dec(Sh, L, t + 1);
  float* dec_out = Win::dec(Sh, L, t);
  const float* cin = scale_in + bh * L;
  auto lam_of = [&](int l) { return lam ? lam[bh * L + l] : 1.f; };
  auto level_row = [&](int l, int x) { return Sh + ((int64_t)l * DV + row0 + 16 * x) * DK; };

  float qv[NPT], kv[NPT];
  RP::template load<sizeof(T)>(q + bh * DK, c, qv);
  RP::template load<sizeof(T)>(k + bh * DK, c, kv);
  const float alpha = expf(log_alpha[bh]);

  // levels that carry over, decayed by alpha_t; the first batch's rows are requested before the window
  const int p = MERGE ? __builtin_ctzll((unsigned long long)t) : LOGW - 1;
  int64_t rest = t >> (p + 1);
  int l0 = p + 2;
  // Levels decayed to nothing (scale 0) are not read.  1024 heads, d = 128, log alpha about -3, positions 3968 ..
  // 4095: 76.9 -> 25.7 us a step; where every level counts, the wait for the scales costs nothing (77.3, 77.4).
  // Masking only the levels after the first batch: 26.9, and at 256 heads 19.4 against 14.3.
  const int lane = tid & 63;
  const float cl_lane = cin[lane < L ? lane : 0];
  rest &= (int64_t)(__ballot(lane < L && cl_lane != 0.f) >> l0);
  // Tokens decayed to nothing are left out like such levels, whatever they hold (0 times a value that is not finite
  // would stay): of the window merged below, those before s0 (the decays do not fall from token to token).
  int s0 = 0;
  if constexpr (MERGE) {
    const uint64_t live = __ballot(lane < W && dec_in[lane < W ? lane : 0] != 0.f);
    s0 = live ? __builtin_ctzll(live) : W;
  }
  LevelBatch<KB> lv;
  float x[KB][RB][NPT];
  auto load_levels = [&]() {
    lv.next(rest, l0);
#pragma unroll
    for (int b = 0; b < KB; ++b)
      if (b < lv.n)
#pragma unroll
        for (int y = 0; y < RB; ++y) RP::load(level_row(lv.l[b], y), c, x[b][y]);
  };
  load_levels();

  // this lane's tokens of the window: v at the rows, requested with the levels
  constexpr int WV = (W + 15) / 16;
  float vw[RB][WV];
#pragma unroll
  for (int y = 0; y < RB; ++y)
#pragma unroll
    for (int u = 0; u < WV; ++u) {
      const int s = window_slot(c, u, i);
      vw[y][u] = s >= 0 ? to_f32(win.v[s * DV + row0 + 16 * y]) : 0.f;
    }
  float acc[RB];  // this thread's part of the rows' outputs
#pragma unroll
  for (int y = 0; y < RB; ++y) acc[y] = 0.f;
  if constexpr (MERGE) {
    // level p+1 <- levels LOGW+1 .. p and the full window
    const Win full(Sh, L, (t >> LOGW) - 1);
    float m[RB][NPT];
#pragma unroll
    for (int y = 0; y < RB; ++y)
#pragma unroll
      for (int e = 0; e < NPT; ++e) m[y][e] = 0.f;
    auto add_token = [&](int s) {
      const float d = dec_in[s];
      float ks[NPT];
      RP::load(full.k + s * DK, c, ks);
#pragma unroll
      for (int y = 0; y < RB; ++y) {
        const float vs = d * to_f32(full.v[s * DV + row0 + 16 * y]);
#pragma unroll
        for (int e = 0; e < NPT; ++e) m[y][e] += vs * ks[e];
      }
    };
    if (s0 == 0) {
#pragma unroll 4
      for (int s = 0; s < W; ++s) add_token(s);
    } else {
      for (int s = s0; s < W; ++s) add_token(s);
    }
    for (int l = LOGW + 1; l <= p; ++l) {
      const float cl = cin[l];
      if (cl == 0.f) continue;
#pragma unroll
      for (int y = 0; y < RB; ++y) {
        float z[NPT];
        RP::load(level_row(l, y), c, z);
#pragma unroll
        for (int e = 0; e < NPT; ++e) m[y][e] += cl * z[e];
      }
    }
    const float w = lam_of(p + 1) * alpha;
#pragma unroll
    for (int y = 0; y < RB; ++y) {
      RP::store(level_row(p + 1, y), c, m[y]);
      acc[y] += w * RP::dot(m[y], qv);
    }
  } else {
    // the window's tokens: p_s = lambda^(l(t,s)) decay (k_s . q_t), 16 lanes per token
    for (int s = r; s < i; s += 16) {
      float ks[NPT];
      RP::load(win.k + s * DK, c, ks);
      const float a = sum16(RP::dot(ks, qv));
      if (c == 0) {
        const float d0 = dec_in[s], d = d0 * alpha, w = lam_of(bitlen(uint32_t(i ^ s))) * d * a + 0.f;
        p_s[s] = d0 != 0.f ? w : kLeftOut;
        if (blockIdx.x == 0) dec_out[s] = d;
      }
    }
    __syncthreads();
  }
  while (lv.n) {
#pragma unroll
    for (int b = 0; b < KB; ++b)
      if (b < lv.n) {
        const float w = lam_of(lv.l[b]) * cin[lv.l[b]] * alpha;
#pragma unroll
        for (int y = 0; y < RB; ++y) acc[y] += w * RP::dot(x[b][y], qv);
      }
    load_levels();
  }
  // the token itself, level 0: v_t[row] (k_t . q_t)
  const float kq = sum16(RP::dot(kv, qv));
  float pw[WV];
  if constexpr (!MERGE)
#pragma unroll
    for (int u = 0; u < WV; ++u) {
      const int s = window_slot(c, u, i);
      pw[u] = s >= 0 ? p_s[s] : kLeftOut;
      const bool out = __float_as_uint(pw[u]) == __float_as_uint(kLeftOut);
#pragma unroll
      for (int y = 0; y < RB; ++y) vw[y][u] = out ? 0.f : vw[y][u];
    }
#pragma unroll
  for (int y = 0; y < RB; ++y) {
    const int row = row0 + 16 * y;
    float a = acc[y];
    if constexpr (!MERGE)
#pragma unroll
      for (int u = 0; u < WV; ++u) a += pw[u] * vw[y][u];
    a = sum16(a);
    if (c == 0) o[bh * DV + row] = from_f32<T>(a + lam_of(0) * to_f32(v[bh * DV + row]) * kq);
  }

  // the next step's scales (the other parity buffer) and the token's window slot
  if (blockIdx.x == 0) {
    float* cout = scale_out + bh * L;
    for (int l = tid; l < L; l += kDecodeThreads) {
      // after token t level l >= 1 holds tokens iff bit l - 1 of t is set
      const bool held = l > LOGW && ((t >> (l - 1)) & 1);
      cout[l] = !held ? 0.f : (MERGE && l == p + 1) ? alpha : cin[l] * alpha;
    }
    for (int e = tid; e < DK; e += kDecodeThreads) win.k[i * DK + e] = from_f32<Row>(to_f32(k[bh * DK + e]));
    for (int e = tid; e < DV; e += kDecodeThreads) win.v[i * DV + e] = from_f32<Row>(to_f32(v[bh * DV + e]));
    if (tid == 0) dec_out[i] = 1.f;
  }
}

// ---------------------------------------------------------------------------------------------
// Log-linear Gated DeltaNet decoding.  The transition A_t = alpha_t (I - beta_t k_t k_t^T) acts on every
// level; a token's part of the output is lambda_t^(l(t,s)) beta_s (k_s . A_{s+1} .. A_t q_t) v_s.  With
// the window's tokens kept as rows (as above), the query is carried back through them instead of the
// levels forward: with w_s = k_s . q^(s), q^(t) = q_t, q^(s-1) = q^(s) - beta_s w_s k_s (decays aside),
//     w_s = k_s . q_t - sum_{r > s} beta_r w_r (k_r . k_s),
// a triangular solve with the window's Gram matrix (one wave, one lane per token), and every level above
// the window is read once with q~ = decay (q_t - sum_s beta_s w_s k_s), its matrix unchanged.  Applying
// the transitions to every level at each token instead reads and writes all of them each step.  The
// step that opens the next window (t % W == 0) applies the full window's W transitions to every level,
// row by row in registers, adds the window's own tokens to the merged one and writes them all.
// 1024 heads, d = 128, bf16, W = 32, positions 2976 .. 3039: 208 -> 72 us a step on average, the merges in it 193,
// where the worst step that rewrites every level took 263 (decode_log_window: other batches).  Registers bound
// the waves in flight: the Gram rows in registers instead of LDS, or spilling to 80 or 64 of them, cost 7 to
// 60 % of the step.
// ---------------------------------------------------------------------------------------------
template <typename T, int DK, int DV, int LOGW, int RB>
__global__ __launch_bounds__(kDecodeThreads) void k_gdn_decode_step(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, const float* __restrict__ log_alpha,
    const float* __restrict__ beta, const float* __restrict__ lam, T* __restrict__ o, float* __restrict__ S, int64_t t,
    int L) {
  typedef RowPart<DK> RP;
  typedef WindowRow<T, DK, DV> Row;
  typedef DecodeWindow<Row, DK, DV, LOGW> Win;
  constexpr int NPT = RP::NPT, W = Win::W;
  constexpr int KB = RB >= 4 ? 1 : 4;                 // levels loaded together
  constexpr int QP = kDecodeThreads / DK < W ? kDecodeThreads / DK : W;  // partial sums of q~ per column
  __shared__ __attribute__((aligned(16))) Row k_s[W * DK];
  __shared__ __attribute__((aligned(16))) float qp_s[QP * DK];
  __shared__ float a_s[W], g_s[W], cf_s[W], p_s[W], gr_s[W * W + 64], db_s;  // gr_s: 64 lanes read a row
  const int64_t bh = blockIdx.y;
  const int tid = threadIdx.x, r = tid >> 4, c = tid & 15;
  const int row0 = blockIdx.x * 16 * RB + r;
  const int i = (int)(t & (W - 1));
  float* Sh = S + bh * (int64_t)L * DV * DK;
  const Win win(Sh, L, t >> LOGW);
  const int cap = Win::cap(L);
  const float* dec_in = Win::dec(Sh, L, t + 1);
  float* dec_out = Win::dec(Sh, L, t);
  auto lam_of = [&](int l) { return lam ? lam[bh * L + l] : 1.f; };
  auto level_row = [&](int l, int x) { return Sh + ((int64_t)l * DV + row0 + 16 * x) * DK; };

  float qv[NPT], kv[NPT];
  RP::template load<sizeof(T)>(q + bh * DK, c, qv);
  RP::template load<sizeof(T)>(k + bh * DK, c, kv);
  const float alpha = expf(log_alpha[bh]), bt = beta[bh];

  int64_t rest = t >> LOGW;
  int l0 = LOGW + 1;
  LevelBatch<KB> lv;
  float x[KB][RB][NPT];
  auto load_levels = [&]() {
    lv.next(rest, l0);
#pragma unroll
    for (int b = 0; b < KB; ++b)
      if (b < lv.n)
#pragma unroll
        for (int y = 0; y < RB; ++y) RP::load(level_row(lv.l[b], y), c, x[b][y]);
  };
  load_levels();

  // this lane's tokens of the window: v at the rows, requested with the levels
  constexpr int WV = (W + 15) / 16;
  float vw[RB][WV];
#pragma unroll
  for (int y = 0; y < RB; ++y)
#pragma unroll
    for (int u = 0; u < WV; ++u) {
      const int s = window_slot(c, u, i);
      vw[y][u] = s >= 0 ? to_f32(win.v[s * DV + row0 + 16 * y]) : 0.f;
    }
  for (int e = tid; e < i * cap; e += kDecodeThreads) gr_s[e] = win.gram[e];  // its first i rows
  // wave 0: what the triangular solve needs besides, one token per lane
  float bs = bt, dec = 1.f, lw = 0.f;
  if (tid < i) {
    bs = win.beta[tid];
    dec = dec_in[tid] * alpha;
  }
  if (tid <= i) lw = lam_of(bitlen(uint32_t(i ^ tid)));

  // ---- window: k_s . q_t and k_s . k_t for its tokens and the new one
  for (int s = r; s <= i; s += 16) {
    float ks[NPT];
    if (s < i) RP::load(win.k + s * DK, c, ks);
    else
#pragma unroll
      for (int e = 0; e < NPT; ++e) ks[e] = kv[e];
    RP::store(k_s + s * DK, c, ks);
    const float a = sum16(RP::dot(ks, qv)), g = sum16(RP::dot(ks, kv));
    if (c == 0) {
      a_s[s] = a;
      g_s[s] = g;
    }
  }
  __syncthreads();
  if (tid < 64) {
    const float g = tid < i ? g_s[tid] : 0.f;
    float w = tid <= i ? a_s[tid] : 0.f;
    w -= bt * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), i)) * g;
#pragma unroll
    for (int s = W - 1; s >= 0; --s)
      if (s < i)
        w -= __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bs * w), s)) * (tid < s ? gr_s[s * cap + tid] : 0.f);
    if (tid < W) {
      cf_s[tid] = tid <= i ? bs * w : 0.f;
      p_s[tid] = lw * dec * bs * w;
    }
    const float db = i ? dec_in[cap] * alpha : alpha;  // decay of the whole window
    if (tid == 0) db_s = db;
    if (blockIdx.x == 0 && tid <= i) {
      dec_out[tid] = dec;
      if (tid < i) win.gram[i * cap + tid] = g;
      if (tid == i) {
        win.beta[i] = bt;
        win.alpha[i] = alpha;
        dec_out[cap] = db;
      }
    }
  }
  __syncthreads();
  if (QP * DK == kDecodeThreads || tid < QP * DK) {
    const int n = tid % DK;
    float a = 0.f;
#pragma unroll
    for (int u = 0; u < W / QP; ++u) {  // past token i: weight 0
      const int s = tid / DK + QP * u;
      a += cf_s[s] * to_f32(k_s[(s < i ? s : i) * DK + n]);
    }
    qp_s[tid] = a;
  }
  __syncthreads();
  float qt[NPT];
  {
    const float db = db_s;
#pragma unroll
    for (int e = 0; e < NPT; ++e) qt[e] = qv[e];
#pragma unroll
    for (int y = 0; y < QP; ++y) {
      float z[NPT];
      RP::load(qp_s + y * DK, c, z);
#pragma unroll
      for (int e = 0; e < NPT; ++e) qt[e] -= z[e];
    }
#pragma unroll
    for (int e = 0; e < NPT; ++e) qt[e] *= db;
  }

  // ---- levels above the window, read with q~
  float acc[RB];
#pragma unroll
  for (int y = 0; y < RB; ++y) acc[y] = 0.f;
  while (lv.n) {
#pragma unroll
    for (int b = 0; b < KB; ++b)
      if (b < lv.n) {
        const float w = lam_of(lv.l[b]);
#pragma unroll
        for (int y = 0; y < RB; ++y) acc[y] += w * RP::dot(x[b][y], qt);
      }
    load_levels();
  }
#pragma unroll
  for (int y = 0; y < RB; ++y) {
    const int row = row0 + 16 * y;
    float a = acc[y];
#pragma unroll
    for (int u = 0; u < WV; ++u)
      if (const int s = window_slot(c, u, i); s >= 0) a += p_s[s] * vw[y][u];
    a = sum16(a);
    if (c == 0) o[bh * DV + row] = from_f32<T>(a + p_s[i] * to_f32(v[bh * DV + row]));
  }
  if (blockIdx.x == 0) {
    for (int e = tid; e < DK; e += kDecodeThreads) win.k[i * DK + e] = from_f32<Row>(to_f32(k[bh * DK + e]));
    for (int e = tid; e < DV; e += kDecodeThreads) win.v[i * DV + e] = from_f32<Row>(to_f32(v[bh * DV + e]));
  }
}

// Token t with t % W == 0, t > 0: every level through the full window's transitions (row x of a level:
// x <- x - beta_s (x . k_s) k_s for s in order, then the window's decay), then token t as the first of
// its window.  The merged level p + 1 is the sum of levels LOGW + 1 .. p before them and of the window's
// tokens, which enter in turn (x <- alpha_s (x - beta_s (x . k_s) k_s) + beta_s v_s[row] k_s).
// 8 lanes per row: the 2 DK / 8 multiplications and additions of a transition outweigh the lanes' sum
// (16 lanes: 414 us for 6 levels of 1024 heads, d = 128, W = 32; 8: 290).
constexpr int kMergeLanes = 8;

template <typename T, int DK, int DV, int LOGW>
__global__ __launch_bounds__(DV * kMergeLanes < kDecodeThreads ? DV * kMergeLanes : kDecodeThreads) void
k_gdn_decode_merge(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                   const float* __restrict__ log_alpha, const float* __restrict__ beta, const float* __restrict__ lam,
                   T* __restrict__ o, float* __restrict__ S, int64_t t, int L) {
  typedef RowPart<DK, kMergeLanes> RP;
  typedef WindowRow<T, DK, DV> Row;
  typedef DecodeWindow<Row, DK, DV, LOGW> Win;
  constexpr int NPT = RP::NPT, W = Win::W, NB = 4;
  constexpr int NTH = DV * kMergeLanes < kDecodeThreads ? DV * kMergeLanes : kDecodeThreads, ROWS = NTH / kMergeLanes;
  __shared__ __attribute__((aligned(16))) float k_s[W * DK];
  __shared__ float bv_s[W * ROWS], b_s[W], al_s[W];
  const int64_t bh = blockIdx.y;
  const int tid = threadIdx.x, r = tid / kMergeLanes, c = tid % kMergeLanes;
  const int row = blockIdx.x * ROWS + r;
  float* Sh = S + bh * (int64_t)L * DV * DK;
  const Win full(Sh, L, (t >> LOGW) - 1), win(Sh, L, t >> LOGW);
  auto lam_of = [&](int l) { return lam ? lam[bh * L + l] : 1.f; };
  auto level_row = [&](int l) { return Sh + ((int64_t)l * DV + row) * DK; };
  const int p = __builtin_ctzll((unsigned long long)t);

  for (int s = r; s < W; s += ROWS) {
    float ks[NPT];
    RP::load(full.k + s * DK, c, ks);
    RP::store(k_s + s * DK, c, ks);
  }
  for (int e = tid; e < W * ROWS; e += NTH)
    bv_s[e] = full.beta[e / ROWS] * to_f32(full.v[e / ROWS * DV + blockIdx.x * ROWS + e % ROWS]);
  for (int s = tid; s < W; s += NTH) {
    b_s[s] = full.beta[s];
    al_s[s] = full.alpha[s];
  }
  float qt[NPT], kv[NPT];  // q~ = alpha_t (q - beta_t (k . q) k)
  RP::template load<sizeof(T)>(q + bh * DK, c, qt);
  RP::template load<sizeof(T)>(k + bh * DK, c, kv);
  const float alpha = expf(log_alpha[bh]), bt = beta[bh];
  const float kq = sum8(RP::dot(kv, qt));
#pragma unroll
  for (int e = 0; e < NPT; ++e) qt[e] = alpha * (qt[e] - bt * kq * kv[e]);
  const float dw = Win::dec(Sh, L, t + 1)[Win::cap(L)];  // decay of the full window

  // levels lowest first: the merged one, then the carried ones, NB at a time
  float acc = 0.f;
  int64_t rest = t >> (p + 1);
  int l0 = p + 2;
  LevelBatch<NB> lv;
  float x[NB][NPT];
  auto load_levels = [&]() {
    lv.next(rest, l0);
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (b < lv.n) RP::load(level_row(lv.l[b]), c, x[b]);
  };
  load_levels();
  {
    float m[NPT];
#pragma unroll
    for (int e = 0; e < NPT; ++e) m[e] = 0.f;
    for (int l = LOGW + 1; l <= p; ++l) {
      float z[NPT];
      RP::load(level_row(l), c, z);
#pragma unroll
      for (int e = 0; e < NPT; ++e) m[e] += z[e];
    }
    __syncthreads();
#pragma unroll 2
    for (int s = 0; s < W; ++s) {
      float ks[NPT];
      RP::load(k_s + s * DK, c, ks);
      const float al = al_s[s];
      const float y = bv_s[s * ROWS + r] - al * b_s[s] * sum8(RP::dot(m, ks));
#pragma unroll
      for (int e = 0; e < NPT; ++e) m[e] = al * m[e] + y * ks[e];
    }
    RP::store(level_row(p + 1), c, m);
    acc += lam_of(p + 1) * RP::dot(m, qt);
  }
  while (lv.n) {
#pragma unroll
    for (int b = 0; b < NB; ++b)  // a short batch: the rows past it are not used
      if (b >= lv.n)
#pragma unroll
        for (int e = 0; e < NPT; ++e) x[b][e] = 0.f;
#pragma unroll 2
    for (int s = 0; s < W; ++s) {
      float ks[NPT];
      RP::load(k_s + s * DK, c, ks);
      const float bs = b_s[s];
      float y[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) y[b] = -bs * sum8(RP::dot(x[b], ks));
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < NPT; ++e) x[b][e] += y[b] * ks[e];
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (b < lv.n) {
#pragma unroll
        for (int e = 0; e < NPT; ++e) x[b][e] *= dw;
        RP::store(level_row(lv.l[b]), c, x[b]);
        acc += lam_of(lv.l[b]) * RP::dot(x[b], qt);
      }
    load_levels();
  }
  acc = sum8(acc);
  if (c == 0) o[bh * DV + row] = from_f32<T>(acc + lam_of(0) * bt * to_f32(v[bh * DV + row]) * kq);

  if (blockIdx.x == 0) {
    for (int e = tid; e < DK; e += NTH) win.k[e] = from_f32<Row>(to_f32(k[bh * DK + e]));
    for (int e = tid; e < DV; e += NTH) win.v[e] = from_f32<Row>(to_f32(v[bh * DV + e]));
    if (tid == 0) {
      win.beta[0] = bt;
      win.alpha[0] = alpha;
      float* dec_out = Win::dec(Sh, L, t);
      dec_out[0] = 1.f;
      dec_out[Win::cap(L)] = alpha;
    }
  }
}

// Every level kept as a matrix, its transition applied at each token: small batches, whose levels stay in the
// caches.  Level 0 is kept in factored form, f0: beta v and k of the previous token.  Row x of a level takes
// x <- alpha (x - beta (x . k) k) on its own, the split is that of k_gdn_decode_step, and for t >= 1, with
// p = lssb(t), level p + 1 is first the sum of levels 0 .. p.
template <typename T, int DK, int DV>
__global__ __launch_bounds__(kDecodeThreads) void k_gdn_decode_plain(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, const float* __restrict__ log_alpha,
    const float* __restrict__ beta, const float* __restrict__ lam, T* __restrict__ o, float* __restrict__ S,
    const float* __restrict__ f0_in, float* __restrict__ f0_out, int64_t t, int L) {
  typedef RowPart<DK> RP;
  constexpr int NPT = RP::NPT, NB = 4;  // levels loaded together
  const int64_t bh = blockIdx.y;
  const int tid = threadIdx.x, r = tid >> 4, c = tid & 15;
  const int row = blockIdx.x * 16 + r;
  float* Sh = S + bh * (int64_t)L * DV * DK;
  auto lam_of = [&](int l) { return lam ? lam[bh * L + l] : 1.f; };
  auto level_row = [&](int l) { return Sh + ((int64_t)l * DV + row) * DK; };
  float x[NB][NPT];
  LevelBatch<NB> lv;
  int64_t rest = 0;
  int l0 = 0;
  auto load_levels = [&]() {
    lv.next(rest, l0);
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (b < lv.n) RP::load(level_row(lv.l[b]), c, x[b]);
  };

  float qv[NPT], kv[NPT];
  RP::template load<sizeof(T)>(q + bh * DK, c, qv);
  RP::template load<sizeof(T)>(k + bh * DK, c, kv);
  const float alpha = expf(log_alpha[bh]), bt = beta[bh];
  const float kq = sum16(RP::dot(kv, qv));
  float acc = 0.f;  // the row's output (the same in its 16 lanes)
  auto step_level = [&](float (&y)[NPT], int l) {
    const float a = sum16(RP::dot(y, kv)), b = sum16(RP::dot(y, qv));
#pragma unroll
    for (int e = 0; e < NPT; ++e) y[e] = alpha * (y[e] - bt * a * kv[e]);
    RP::store(level_row(l), c, y);
    acc += lam_of(l) * alpha * (b - bt * kq * a);
  };
  if (t > 0) {
    const int p = __builtin_ctzll((unsigned long long)t);
    const float* f = f0_in + bh * (DV + DK);
    const float bv = f[row];
    float m[NPT];
    RP::load(f + DV, c, m);
#pragma unroll
    for (int e = 0; e < NPT; ++e) m[e] *= bv;
    rest = (int64_t(1) << p) - 1;  // levels 1 .. p
    l0 = 1;
    for (load_levels(); lv.n; load_levels())
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (b < lv.n)
#pragma unroll
          for (int e = 0; e < NPT; ++e) m[e] += x[b][e];
    rest = t >> (p + 1);  // the others that hold tokens
    l0 = p + 2;
    load_levels();
    step_level(m, p + 1);
    for (; lv.n; load_levels())
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (b < lv.n) step_level(x[b], lv.l[b]);
  }
  if (c == 0) o[bh * DV + row] = from_f32<T>(acc + lam_of(0) * bt * to_f32(v[bh * DV + row]) * kq);

  if (blockIdx.x == 0) {
    float* f = f0_out + bh * (DV + DK);
    for (int e = tid; e < DV; e += kDecodeThreads) f[e] = bt * to_f32(v[bh * DV + e]);
    for (int e = tid; e < DK; e += kDecodeThreads) f[DV + e] = to_f32(k[bh * DK + e]);
  }
}

// Zero-fills n floats (the decode state before its first token).
__global__ void k_zero_f32(float* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

// Rows of d_v per workgroup, in 16s: 4 once that still gives every CU several workgroups (a window's
// scores are formed once per workgroup), else 1, so that a small batch spreads over the chip.
// d = 128, W = 32, 16 against 64 rows: 53.7 / 50.0 us and 29.1 / 25.9 us (Mamba-2, 1024 and 512 heads), 80.3 / 61.6
// and 44.0 / 31.7 us (Gated DeltaNet); 256 heads or fewer keep 16.
template <int DV>
bool decode_wide(int64_t BH) {
  return DV % 64 == 0 && BH * (DV / 64) >= 1024;
}

// log2 of the window, the same for every step of a state (it depends on the state's sizes alone).  A longer window
// merges less often and reads more rows meanwhile; a merge of W tokens is a chain as long as W that a small
// batch waits for (its levels stay in the caches, where reading them costs little).  So 8 tokens below 2^21
// matrix entries per level (BH d_k d_v), 32 where the levels come from memory, 16 between.  Mean of positions 2976 ..
// 3039 and worst step, us, W = 8 / 16 / 32, d = 128: Mamba-2 4.7 / 4.7 / 5.1 and 7.9 / 8.8 / 10.2 (16 heads),
// 18.0 / 17.6 / 18.7 and 28 / 31 / 37 (256), 75 / 67 / 62 and 113 / 105 / 132 (1024); Gated DeltaNet 7.8 / 7.6 / 8.7 and
// 20 / 25 / 28 (64), 22.3 / 21.8 / 24.0 and 43 / 53 / 61 (256), 88 / 76 / 72 and 149 / 189 / 193 (1024).  0: Gated DeltaNet
// without a window (k_gdn_decode_plain) up to 2^19 entries (2^18 for d = 16); without and with W = 8, positions 0 .. 31,
// 96 .. 159, 2976 .. 3039 and the last's worst step, d = 128: 4.0, 4.4, 5.7, 9.0 us and 4.8, 5.3, 6.3, 16 (16 heads);
// 5.2, 6.5, 10.1, 15.6 and 5.4, 6.2, 7.9, 19.4 (64 heads); 128 x 64: 4.5, 5.3, 6.9, 10.7 and 5.0, 5.6, 6.9, 19.2 (64 heads).
template <int DK, int DV>
int decode_log_window(int64_t BH, bool gdn) {
  const int64_t entries = BH * DK * DV;
  if (gdn && entries <= (int64_t(1) << (DK == 16 ? 18 : 19))) return 0;
  if (DK == 16) return 3;  // a row is not much smaller than a matrix
  return entries < (int64_t(1) << 21) ? 3 : entries < (int64_t(1) << (gdn ? 24 : 23)) ? 4 : 5;
}
// Calls f with the window's log2 as a compile-time constant.
template <int DK, int DV, typename F>
void with_log_window(int64_t BH, bool gdn, F f) {
  const int log = decode_log_window<DK, DV>(BH, gdn);
  if (log == 0) return f(std::integral_constant<int, 0>{});
  if constexpr (DK != 16) {
    if (log == 4) return f(std::integral_constant<int, 4>{});
    if (log == 5) return f(std::integral_constant<int, 5>{});
  }
  f(std::integral_constant<int, 3>{});
}

template <typename T, int DK, int DV>
hipError_t launch_decode(const void* q, const void* k, const void* v, const float* log_alpha, const float* lambda,
                         void* o, void* state, int64_t t, int64_t B, int64_t H, int L, hipStream_t st) {
  const DecodeLayout d = decode_layout(B, H, DK, DV, L);
  char* base = static_cast<char*>(state);
  const int64_t BH = B * H;
  float* S = reinterpret_cast<float*>(base + d.S);
  float* scale = reinterpret_cast<float*>(base + d.scale);
  const int par = (int)(t & 1);
  constexpr int RW = DV % 64 == 0 ? 4 : 1;
  auto launch = [&](auto kernel, int rb) {
    hipLaunchKernelGGL(kernel, dim3(DV / (16 * rb), (unsigned)BH), dim3(kDecodeThreads), 0, st, (const T*)q,
                       (const T*)k, (const T*)v, log_alpha, lambda, (T*)o, S, scale + (1 - par) * BH * L,
                       scale + par * BH * L, t, L);
  };
  with_log_window<DK, DV>(BH, false, [&](auto log) {
    constexpr int LOGW = decltype(log)::value > 3 ? decltype(log)::value : 3;
    if (t > 0 && t % (1 << LOGW) == 0) launch(k_decode_step<T, DK, DV, LOGW, 1, true>, 1);
    else if (LOGW > 3 && decode_wide<DV>(BH)) launch(k_decode_step<T, DK, DV, LOGW, (LOGW > 3 ? RW : 1), false>, RW);
    else launch(k_decode_step<T, DK, DV, LOGW, 1, false>, 1);
  });
  return hipGetLastError();
}

template <typename T, int DK, int DV>
hipError_t launch_gdn_decode(const void* q, const void* k, const void* v, const float* log_alpha, const float* beta,
                             const float* lambda, void* o, void* state, int64_t t, int64_t B, int64_t H, int L,
                             hipStream_t st) {
  const DecodeLayout d = decode_layout(B, H, DK, DV, L);
  const int64_t BH = B * H;
  float* S = reinterpret_cast<float*>(static_cast<char*>(state) + d.S);
  constexpr int RW = DV % 64 == 0 ? 4 : 1;
  auto launch = [&](auto kernel, int threads, int rows) {  // rows of d_v per workgroup
    hipLaunchKernelGGL(kernel, dim3(DV / rows, (unsigned)BH), dim3(threads), 0, st, (const T*)q, (const T*)k,
                       (const T*)v, log_alpha, beta, lambda, (T*)o, S, t, L);
  };
  constexpr int MT = DV * kMergeLanes < kDecodeThreads ? DV * kMergeLanes : kDecodeThreads;
  with_log_window<DK, DV>(BH, true, [&](auto log) {
    constexpr int LOGW = decltype(log)::value;
    if constexpr (LOGW == 0) {
      float* f0 = reinterpret_cast<float*>(static_cast<char*>(state) + d.f0);
      const int64_t par = t & 1, n = BH * (DV + DK);
      hipLaunchKernelGGL((k_gdn_decode_plain<T, DK, DV>), dim3(DV / 16, (unsigned)BH), dim3(kDecodeThreads), 0, st,
                         (const T*)q, (const T*)k, (const T*)v, log_alpha, beta, lambda, (T*)o, S, f0 + (1 - par) * n,
                         f0 + par * n, t, L);
    } else if (t > 0 && t % (1 << LOGW) == 0) {
      launch(k_gdn_decode_merge<T, DK, DV, LOGW>, MT, MT / kMergeLanes);
    } else if (LOGW > 3 && decode_wide<DV>(BH)) {
      launch(k_gdn_decode_step<T, DK, DV, LOGW, (LOGW > 3 ? RW : 1)>, kDecodeThreads, 16 * RW);
    } else {
      launch(k_gdn_decode_step<T, DK, DV, LOGW, 1>, kDecodeThreads, 16);
    }
  });
  return hipGetLastError();
}

hipError_t launch_decode_init(void* state, int64_t B, int64_t H, int64_t dk, int64_t dv, int L, hipStream_t st) {
  const DecodeLayout d = decode_layout(B, H, dk, dv, L);
  // the scales and level-0 factors of both parities.  The rest needs no clearing: a step reads the levels that
  // hold tokens by the bits of t (of Mamba-2 those whose scale is nonzero), and rows that earlier steps wrote
  float* p = reinterpret_cast<float*>(static_cast<char*>(state) + d.scale);
  const int64_t n = (d.total - d.scale) / 4;
  hipLaunchKernelGGL(k_zero_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

typedef hipError_t (*DecodeLaunch)(const void*, const void*, const void*, const float*, const float*, void*, void*,
                                   int64_t, int64_t, int64_t, int, hipStream_t);
typedef hipError_t (*GdnDecodeLaunch)(const void*, const void*, const void*, const float*, const float*, const float*,
                                      void*, void*, int64_t, int64_t, int64_t, int, hipStream_t);
struct DecodeEntry {
  int dtype, dk, dv;
  DecodeLaunch launch;
  GdnDecodeLaunch gdn_launch;
};

#define LL_DECODE_SHAPES(X) \
  X(float, 16, 16)          \
  X(float, 64, 64)          \
  X(__bf16, 64, 64)         \
  X(__bf16, 128, 64)        \
  X(__bf16, 128, 128)

const DecodeEntry* decode_table(int* n) {
#define LL_ENTRY(T, DK, DV) \
  {std::is_same<T, float>::value ? 0 : 1, DK, DV, &launch_decode<T, DK, DV>, &launch_gdn_decode<T, DK, DV>},
  static const DecodeEntry table[] = {LL_DECODE_SHAPES(LL_ENTRY)};
#undef LL_ENTRY
  *n = sizeof(table) / sizeof(table[0]);
  return table;
}

}  // namespace ll

namespace {
const ll::DecodeEntry* find_decode(int32_t dtype, int64_t dk, int64_t dv) {
  int n = 0;
  const ll::DecodeEntry* t = ll::decode_table(&n);
  for (int i = 0; i < n; ++i)
    if (t[i].dtype == dtype && t[i].dk == dk && t[i].dv == dv) return &t[i];
  return nullptr;
}

ll_status check_decode(int64_t B, int64_t H, int64_t d_k, int64_t d_v, int32_t L, int32_t dtype) {
  if (B < 1 || H < 1 || d_k < 1 || d_v < 1 || L < 1) return LL_ERR_BAD_SHAPE;
  if (dtype != LL_F32 && dtype != LL_BF16) return LL_ERR_UNSUPPORTED;
  if (L > ll::kDecodeMaxLevels || B * H > 65535 || !find_decode(dtype, d_k, d_v)) return LL_ERR_UNSUPPORTED;
  return LL_OK;
}
}  // namespace

extern "C" {

size_t ll_decode_state_bytes(int64_t B, int64_t H, int64_t d_k, int64_t d_v, int32_t L) {
  if (B < 1 || H < 1 || d_k < 1 || d_v < 1 || L < 1) return 0;
  return (size_t)ll::decode_layout(B, H, d_k, d_v, L).total;
}

ll_status ll_mamba2_decode_init(void* state, size_t state_bytes, int64_t B, int64_t H, int64_t d_k, int64_t d_v,
                                int32_t L, int32_t dtype, void* stream) {
  if (!state) return LL_ERR_NULL_ARG;
  const ll_status s = check_decode(B, H, d_k, d_v, L, dtype);
  if (s != LL_OK) return s;
  if (state_bytes < (size_t)ll::decode_layout(B, H, d_k, d_v, L).total ||
      (reinterpret_cast<uintptr_t>(state) & 255))
    return LL_ERR_WORKSPACE;
  return ll::launch_decode_init(state, B, H, d_k, d_v, L, static_cast<hipStream_t>(stream)) == hipSuccess
             ? LL_OK
             : LL_ERR_HIP;
}

ll_status ll_mamba2_decode_step(const void* q, const void* k, const void* v, const float* log_alpha,
                                const float* lambda, void* o, void* state, size_t state_bytes, int64_t t, int64_t B,
                                int64_t H, int64_t d_k, int64_t d_v, int32_t L, int32_t dtype, void* stream) {
  if (!q || !k || !v || !log_alpha || !o || !state) return LL_ERR_NULL_ARG;
  const ll_status s = check_decode(B, H, d_k, d_v, L, dtype);
  if (s != LL_OK) return s;
  // token t needs level lssb(t) + 1 < L, i.e. t < 2^(L-1)
  if (t < 0 || (L - 1 < 62 && t >= (int64_t(1) << (L - 1)))) return LL_ERR_BAD_SHAPE;
  if (state_bytes < (size_t)ll::decode_layout(B, H, d_k, d_v, L).total ||
      (reinterpret_cast<uintptr_t>(state) & 255))
    return LL_ERR_WORKSPACE;
  const ll::DecodeEntry* e = find_decode(dtype, d_k, d_v);
  return e->launch(q, k, v, log_alpha, lambda, o, state, t, B, H, L, static_cast<hipStream_t>(stream)) == hipSuccess
             ? LL_OK
             : LL_ERR_HIP;
}

ll_status ll_gdn_decode_init(void* state, size_t state_bytes, int64_t B, int64_t H, int64_t d_k, int64_t d_v,
                             int32_t L, int32_t dtype, void* stream) {
  return ll_mamba2_decode_init(state, state_bytes, B, H, d_k, d_v, L, dtype, stream);
}

ll_status ll_gdn_decode_step(const void* q, const void* k, const void* v, const float* log_alpha, const float* beta,
                             const float* lambda, void* o, void* state, size_t state_bytes, int64_t t, int64_t B,
                             int64_t H, int64_t d_k, int64_t d_v, int32_t L, int32_t dtype, void* stream) {
  if (!q || !k || !v || !log_alpha || !beta || !o || !state) return LL_ERR_NULL_ARG;
  const ll_status s = check_decode(B, H, d_k, d_v, L, dtype);
  if (s != LL_OK) return s;
  if (t < 0 || (L - 1 < 62 && t >= (int64_t(1) << (L - 1)))) return LL_ERR_BAD_SHAPE;
  if (state_bytes < (size_t)ll::decode_layout(B, H, d_k, d_v, L).total ||
      (reinterpret_cast<uintptr_t>(state) & 255))
    return LL_ERR_WORKSPACE;
  const ll::DecodeEntry* e = find_decode(dtype, d_k, d_v);
  return e->gdn_launch(q, k, v, log_alpha, beta, lambda, o, state, t, B, H, L, static_cast<hipStream_t>(stream)) ==
                 hipSuccess
             ? LL_OK
             : LL_ERR_HIP;
}

}  // extern "C"
