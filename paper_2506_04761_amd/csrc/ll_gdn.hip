// Log-linear Gated DeltaNet forward (Sec. 3.4): O = (A (.) M^S (.) M^H) V with
// A = (Q K^T (.) L)(I + diag(beta)(K K^T (.) (L - I)))^{-1} diag(beta), i.e. the recurrence
// S_t = alpha_t S_{t-1} (I - beta_t k_t k_t^T) + beta_t v_t k_t^T read out per Fenwick level.
//
// Chunkwise form (chunks of C tokens; local rows t, s; gamma_t = exp(cl_t) with cl the
// chunk-local inclusive cumulative log-gate; Gamma[t,s] = gamma_t / gamma_s for s <= t):
//   T_G   = (I + diag(beta)(K K^T (.) Gamma (.) (L - I)))^{-1} diag(beta)   (unit-lower solve)
//   W     = T_G diag(gamma) K,   U = T_G V                                   (WY / UT form)
//   P_G   = Q K^T (.) Gamma (.) L
//   intra : O_c = ((P_G T_G) (.) M^H_c) V       -- the chunk's own block of A, level-masked
//   Qc    = diag(gamma) Q - P_G W               -- query seen through the chunk's transitions
//   state : S_end^T = P_z S_start^T + H_z,  P_z = gamma_C I - K~^T W,  H_z = K~^T U,
//           K~ = diag(exp(tot - cl)) K
// An earlier state S (d_v x d_k) reaches row t of the chunk as S q~_t (q~_t = row t of Qc).
// Inter-chunk levels (Sec. 3.3 with the delta-rule transition): per chunk level j the state
// R_j (d_k x d_v) restarts at every chunk z with z % 2^j == 0, absorbs H_z in the source half
// (bit j-1 of z clear) and propagates through P_z everywhere; a chunk with bit j-1 set adds
// lambda_t^(log2 C + j) q~_t^T R_j to its rows, with R_j taken at the chunk's start.
//
// Block tree instead of a sequential scan.  For a block of chunks [a, c) let T = P_{c-1} ... P_a
// (its transition) and A = sum over s in [a, c) of P_{c-1} ... P_{s+1} H_s (its accumulated state);
// the block [a, c) = [a, b) then [b, c) has T = T_hi T_lo and A = T_hi A_lo + A_hi.  The level-j
// state read by chunk z (bit j-1 set) is R_j = T(G_1) ... T(G_{j-1}) A(G_j), with G_j the aligned
// source group of 2^(j-1) chunks ending at ((z >> (j-1)) << (j-1)) and G_1, .. the lower source
// groups of z (its set bits below j-1), the most recent first.  So a chunk reads its levels from
// the lowest set bit up, carrying q~^T through each group's transition: out += lambda^(j) q~^T A(G_j),
// then q~^T <- q~^T T(G_j).  Every source group is the aligned block (level j-1, index
// (z >> (j-1)) - 1) of a binary block tree built level by level.
//
// Pairs.  The leaves of the tree are pairs of chunks: level j = 1 is done where the chunks' factors are at
// hand, and both chunks of a pair read the same nodes above it.  In the kernels below a tree level m
// therefore covers 2^m pairs, and the last pair of an odd chunk count holds one chunk.
//
// Kernels: gdn_pair (one persistent workgroup per compute unit walking its pairs; per chunk the WY solve
// in fp32 by a blocked inversion, all products on MFMA, bf16 operands with fp32 accumulation),
// gdn_combine (one launch per tree level, one workgroup per block and column group) and gdn_read (one
// workgroup per chunk: the level read-out and the final output).
#include <type_traits>

#include "ll_device.hpp"
#include "ll_launch.hpp"

namespace ll {

namespace gdn {

constexpr int kMaxJ = 16;      // inter-chunk levels handled by the read-out (T <= C * 2^16)
typedef __bf16 bf;

// "kfrag" layout of a K x N bf16 matrix X (KR = K rows), in which X is read as the B operand of a
// product Y X: the operand fragment of column tile nt and k step ks (32 rows) is 64 lanes x 8
// elements, lane (n % 16) + 16 ((k % 32) / 8) holding rows k with k % 8 = 0..7 in order.  The same
// bytes are the A-operand fragments of X^T (row tile nt of X^T, k step ks).  Four consecutive rows
// 4i .. 4i + 3 of one column are four consecutive elements.
template <int KR>
__device__ inline int kfrag_idx(int k, int n) {
  return (((n >> 4) * (KR / 32) + (k >> 5)) * 64 + (n & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}

// ---------------------------------------------------------------------------------------------
// Kernel 1: WY solve and products of a pair of chunks.  One workgroup of 8 waves per pair; half `hf`
// (4 waves) takes chunk 2 zp + hf, wave w of a half its 16-row tile w.  Outputs (workspace): per chunk
// Qc [C][DK] bf16 row-major (the query seen through its pair's transitions up to it) and the intra-pair
// output [C][DV] fp32 in the MFMA result layout (16 x 16 tiles, row tile major; lane l of a tile holds
// rows 4 (l / 16) + 0..3 of column l % 16); per pair P [DK][DK] bf16 (kfrag layout for even pairs,
// row-major for odd ones: the two sides of a tree combination) and H [DK][DV] bf16 (kfrag).
//
// A pair's transition is that of 128 tokens, so that the tree and the read-out start at pairs: with
// W_i, U_i the chunks' own WY factors and G = W_1 K~_0^T (64 x 64),
//   W_1' = W_1 P_0 = gamma_0 W_1 - G W_0,   U_1' = U_1 - W_1 H_0 = U_1 - G U_0,
// and the same for Q_1 (its product with H_0 being level log2 C + 1 of chunk 1's rows); then
//   P = gamma_0 gamma_1 I - K~^T [W_0; W_1'],   H = K~^T [U_0; U_1'].
// Against one chunk at a time this halves the nodes written and read and drops a tree level.
//
// Registers carry what one wave both makes and uses: a product formed transposed (rows 4g + r, columns
// lane % 16) is, packed to bf16, an operand of the next one, its k slots in the order of
// frag_down_rows.  LDS per half: K, Q, V (row-major, swizzled; loaded into registers while the previous
// pair's last products run, and stored from there), T_G, and the fp32 blocks of
// L and of the inverse, whose room W takes after the inversion; U takes Q's.
//
// B = 2, H = 16, T = 8192, d = 128: this kernel 184-190 us where the kernel working on single chunks took
// 200-224, and the tree level of 79 us over the chunks, with its 403 MB, is gone; the read-out has one node
// round trip less for half the chunks (160 -> 137 us); the forward 513 -> 396 us.  Bound: bursts of memory
// traffic at one workgroup per compute unit (stamps: of 51 thousand cycles per pair 13 to 20 thousand wait for
// staging or behind stores; the fp32 output between kernels is the largest item, 64 KB per pair), then the
// serial inversion.
//
// ONE (sequences of one or two chunks): no tree and no read-out follow, so P, H, Qc and chunk 1's W_1', U_1' are not
// formed, the output leaves as bf16 rows at once, and where sequences have one chunk the halves take one each.
// T = 64 / 128, d = 128: 12.5 / 14.3 us (8 heads), 14.4 / 32.2 us (512), with everything formed and read out 21.2 / 21.6 and
// 47.8 / 57.2 us; one chunk per workgroup took 17.8 / 20.0 and 36.6 / 69.3.
// ---------------------------------------------------------------------------------------------
template <int DK, int DV>
struct PairHalf {  // LDS of one half
  static constexpr int C = 64;
  __attribute__((aligned(16))) bf k[C * DK];
  __attribute__((aligned(16))) bf q[C * (DK > DV ? DK : DV)];  // Q, then U (own rows of each wave)
  __attribute__((aligned(16))) bf v[C * DV];
  __attribute__((aligned(16))) bf z[C * C];                    // T_G, row-major swizzled
  union {
    __attribute__((aligned(16))) float lx[2][10 * 256];        // blocks (i, j), j <= i, of L and of (I + L)^-1
    __attribute__((aligned(16))) bf w[C * DK];                 // W
  };
  float cl[C], gm[C], dc[C], bt[C];  // cumulative log2-gates, exp2 of them, decay to the chunk's end, beta
};

// Two 16 x 16 results packed to bf16 (lane: rows 4g .. 4g + 3 of column lane % 16), joined to 16-byte pieces:
// lanes of even g receive rows 4g .. 4g + 7 of x, lanes of odd g rows 4(g - 1) .. 4g + 3 of y, so that
// each lane stores one whole piece (8-byte stores halve the lines a store instruction completes).
__device__ inline bf16x8 pair_rows(bf16x4 x, bf16x4 y) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  const u32x2 a = __builtin_bit_cast(u32x2, x), b = __builtin_bit_cast(u32x2, y);
  const auto p0 = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto p1 = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  return __builtin_bit_cast(bf16x8, u32x4{p0[0], p1[0], p0[1], p1[1]});
}

// Entry (r, c) of a 16 x 16 fp32 block whose 4-entry pieces are XOR-swizzled by row.
__device__ inline int blk_at(int r, int c) { return r * 16 + ((((c >> 2) ^ (r >> 1)) & 3) << 2) + (c & 3); }
__device__ inline int blk(int i, int j) { return (i * (i + 1) / 2 + j) * 256; }

template <int DK, int DV, bool HAS_LAMBDA, bool ONE>
__global__ __launch_bounds__(512, 2) void k_gdn_pair(const bf* __restrict__ q, const bf* __restrict__ k,
                                                     const bf* __restrict__ v, const float* __restrict__ log_alpha,
                                                     const float* __restrict__ beta, const float* __restrict__ lam,
                                                     bf* __restrict__ qc_out, bf* __restrict__ pz_out,
                                                     bf* __restrict__ hz_out, float* __restrict__ oin_out,
                                                     bf* __restrict__ o_out, int64_t Tlen, int H, int L,
                                                     int64_t npairs, int64_t nseq) {
  using M = Mfma<bf>;
  typedef M::frag frag;
  constexpr int C = 64, KS = DK / 32, KT = DK / 16, VT = DV / 16, NL = 8;  // NL: levels inside a pair
  static_assert(DK == DV, "U takes Q's place");
  __shared__ PairHalf<DK, DV> half_s[2];
  __shared__ float lam_s[HAS_LAMBDA ? 2 * C * NL : 1];

  const int64_t N = Tlen / C, N2 = (N + 1) / 2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), hf = wave >> 2, w = wave & 3;
  PairHalf<DK, DV>&S = half_s[hf], &S0 = half_s[0], &S1 = half_s[1];
  bf* k_s = S.k;
  bf* z_s = S.z;
  float *l_s = S.lx[0], *x_s = S.lx[1];
  float* lam_h = lam_s + (HAS_LAMBDA ? hf * C * NL : 0);
  auto zero4 = [] { return f32x4{0.f, 0.f, 0.f, 0.f}; };
  auto pack = [](f32x4 x) {
    bf16x4 y;
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = static_cast<bf>(x[r]);
    return y;
  };
  auto join = [](bf16x4 lo, bf16x4 hi) { return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7); };

  // A persistent grid (one workgroup per CU, whose LDS allows no second): pairs blockIdx.x,
  // blockIdx.x + gridDim.x, .. in logical order (b, h, pair); the next pair's inputs are loaded into
  // registers while the last products of the current one run.
  struct Where {
    int64_t zp, bh, tok0;
    int h;
    bool valid;  // this half's chunk exists
  };
  auto where = [&](int64_t it) {
    Where x;
    const int64_t work = xcd_remap(it, npairs);
    if (ONE && N == 1) {  // the halves take two sequences
      const int64_t seq = 2 * work + hf;
      x.valid = seq < nseq;
      x.zp = 0;
      x.bh = x.valid ? seq : nseq - 1;
      x.h = (int)(x.bh % H);
      x.tok0 = (x.bh / H) * Tlen;
      return x;
    }
    x.zp = work % N2;
    x.bh = work / N2;
    x.h = (int)(x.bh % H);
    // a sequence of an odd number of chunks: the last pair's second chunk repeats the first one's
    // rows with beta = 0 and no decay (no effect), and stores nothing
    x.valid = 2 * x.zp + hf < N;
    x.tok0 = (x.bh / H) * Tlen + (2 * x.zp + (x.valid ? hf : 0)) * C;
    return x;
  };
  constexpr int CH = DK / 8, PCS = C * CH / 256, NLW = HAS_LAMBDA ? C * NL / 256 : 1;
  bf16x8 kpre[PCS], qpre[PCS], vpre[PCS];  // piece (tid % 256) + 256 e: row piece / CH, 8 columns
  float la_r, bt_r, lam_r[NLW];
  auto load_inputs = [&](const Where& x, int tid) {
    la_r = log_alpha[(x.tok0 + (tid & 63)) * H + x.h];
    bt_r = beta[(x.tok0 + (tid & 63)) * H + x.h];
    if constexpr (HAS_LAMBDA) {
#pragma unroll
      for (int e = 0; e < NLW; ++e) {
        const int y = (tid & 255) + 256 * e, l = y % NL;
        lam_r[e] = lam[((x.tok0 + y / NL) * H + x.h) * L + (l < L ? l : L - 1)];
      }
    }
#pragma unroll
    for (int e = 0; e < PCS; ++e) {
      const int y = (tid & 255) + 256 * e;
      const int64_t at = ((x.tok0 + y / CH) * H + x.h) * DK + 8 * (y % CH);
      kpre[e] = *reinterpret_cast<const bf16x8*>(k + at);
      qpre[e] = *reinterpret_cast<const bf16x8*>(q + at);
      vpre[e] = *reinterpret_cast<const bf16x8*>(v + at);
    }
  };
  Where cur = where(blockIdx.x);
  load_inputs(cur, threadIdx.x);
  for (int64_t it = blockIdx.x; it < npairs; it += gridDim.x) {
  // opaque in every turn: the compiler would otherwise form the many lane-dependent LDS addresses of
  // the body before the loop and spill them
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int64_t zp = cur.zp, bh = cur.bh;
  const bool valid = cur.valid;
  const int64_t cidx = bh * N + 2 * zp + hf;
  if (it != (int64_t)blockIdx.x) __syncthreads();  // the previous pair's readers of LDS are done
#pragma unroll
  for (int e = 0; e < PCS; ++e) {
    const int y = (tid & 255) + 256 * e, at = swz<DK>(y / CH, y % CH);
    *reinterpret_cast<bf16x8*>(S.k + at) = kpre[e];
    *reinterpret_cast<bf16x8*>(S.q + at) = qpre[e];
    *reinterpret_cast<bf16x8*>(S.v + at) = vpre[e];
  }
  if constexpr (HAS_LAMBDA) {
#pragma unroll
    for (int e = 0; e < NLW; ++e) lam_h[(tid & 255) + 256 * e] = lam_r[e];
  }
  if (w == 0) {
    const float cl = wave_inclusive_scan(valid ? la_r * kLog2e : 0.f);
    const float tot = __shfl(cl, C - 1, 64);
    S.cl[lane] = cl;
    S.gm[lane] = fast_exp2(cl);
    S.dc[lane] = fast_exp2(tot - cl);
    S.bt[lane] = valid ? bt_r : 0.f;
  }
  __syncthreads();

  // ---- L[t][s] = beta_t (k_t . k_s) Gamma[t,s], s < t, in 16 x 16 blocks (result layout): the wave's diagonal
  //      block stays in registers, the others (some per wave) go to LDS
  auto form_l = [&](int i, int j) {
    f32x4 acc = zero4();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = M::mma(frag_along_row_swz<DK>(k_s, 16 * i, 4 * ks, lane), frag_along_row_swz<DK>(k_s, 16 * j, 4 * ks, lane), acc);
    const int s = 16 * j + r16;
    const float cs = S.cl[s];
    const f32x4 bt = *reinterpret_cast<const f32x4*>(&S.bt[16 * i + 4 * g]);
    const f32x4 ct = *reinterpret_cast<const f32x4*>(&S.cl[16 * i + 4 * g]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float y = bt[r] * acc[r] * fast_exp2(ct[r] - cs);
      acc[r] = s < 16 * i + 4 * g + r ? y : 0.f;
    }
    return acc;
  };
  auto put_l = [&](int i, int j) {
    const f32x4 y = form_l(i, j);
#pragma unroll
    for (int r = 0; r < 4; ++r) l_s[blk(i, j) + blk_at(4 * g + r, r16)] = y[r];
  };
  const f32x4 ld = form_l(w, w);
  if (w == 0) { put_l(1, 0); put_l(2, 0); }
  if (w == 1) { put_l(2, 1); put_l(3, 0); }
  if (w == 2) put_l(3, 1);
  if (w == 3) put_l(3, 2);
  // ---- X = (I + L)^-1 in 16 x 16 blocks (fp32), T_G = X diag(beta).  Each wave inverts its diagonal block by
  //      forward substitution (lane c of every 16: column c; L_ij from its lane, no LDS: all waves' broadcast
  //      reads of it took 2500 clocks), then the blocks (1,0) and (3,2), then the 32 x 32 block below,
  //      X_21 = -X_22 (L_21 X_11), whose products with diagonal blocks are formed before the barrier.
  auto put_z = [&](int t, int c, float x) { z_s[swz<C>(t, c >> 3) + (c & 7)] = static_cast<bf>(x * S.bt[c]); };
  {
    float x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      f32x4 a = zero4();
#pragma unroll
      for (int j = 0; j < i; ++j)
        a[j & 3] += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ld[i & 3]), 16 * (i >> 2) + j)) * x[j];
      const float acc = ((i == r16) ? 1.f : 0.f) - ((a[0] + a[1]) + (a[2] + a[3]));
      x[i] = (i < r16) ? 0.f : acc;
    }
#pragma unroll
    for (int i = 0; i < 16; i += 4) {  // lane group g stores rows i + g
      const float y0 = x[i], y1 = x[i + 1], y2 = x[i + 2], y3 = x[i + 3];
      const float y = g & 2 ? (g & 1 ? y3 : y2) : (g & 1 ? y1 : y0);
      x_s[blk(w, w) + blk_at(i + g, r16)] = y;
      put_z(16 * w + i + g, 16 * w + r16, y);
    }
  }
  if (!(w & 1))  // zeros of T_G that its products read: blocks (0, 1) and (2, 3)
    *reinterpret_cast<bf16x4*>(z_s + swz<C>(16 * w + r16, 2 * (w + 1) + (g >> 1)) + 4 * (g & 1)) = pack(zero4());
  __syncthreads();
  using MF = Mfma<float>;
  // acc += L_ik X_kj: k slot 4 kk + g
  auto lx_mul = [&](int i, int kb, int j, f32x4 acc) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      acc = MF::mma(l_s[blk(i, kb) + blk_at(r16, 4 * kk + g)], x_s[blk(kb, j) + blk_at(4 * kk + g, r16)], acc);
    return acc;
  };
  // acc += X_ik Y, Y in the result layout (the B operand with k slot 4 g + r)
  auto xy_mul = [&](int i, int kb, f32x4 y, f32x4 acc) {
#pragma unroll
    for (int r = 0; r < 4; ++r) acc = MF::mma(x_s[blk(i, kb) + blk_at(r16, 4 * g + r)], y[r], acc);
    return acc;
  };
  const int bi = 2 + (w >> 1), bj = w & 1;  // the wave's block of X_21
  f32x4 y2 = lx_mul(2, bj, bj, zero4()), y3 = lx_mul(3, bj, bj, zero4());  // L_2j X_jj, L_3j X_jj
  if (!(w & 1)) {
    const f32x4 x = xy_mul(w + 1, w + 1, lx_mul(w + 1, w, w, zero4()), zero4());
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      x_s[blk(w + 1, w) + blk_at(4 * g + r, r16)] = -x[r];
      put_z(16 * (w + 1) + 4 * g + r, 16 * w + r16, -x[r]);
    }
  }
  __syncthreads();
  {
    if (bj == 0) {
      y2 = lx_mul(2, 1, 0, y2);
      y3 = lx_mul(3, 1, 0, y3);
    }
    f32x4 x = xy_mul(bi, 2, y2, zero4());
    if (bi == 3) x += xy_mul(3, 3, y3, zero4());
#pragma unroll
    for (int r = 0; r < 4; ++r) put_z(16 * bi + 4 * g + r, 16 * bj + r16, -x[r]);
  }
  __syncthreads();  // T_G complete; L and X free for W

  const int t_own = 16 * w + r16;  // the wave's row of this lane (columns of the transposed products)
  // ---- P_G^T (rows s, columns t): operand fragments pg (k = s)
  frag pg[2];
  {
    frag qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = frag_along_row_swz<DK>(S.q, 16 * w, 4 * ks, lane);
    const float ct = S.cl[t_own];
    bf16x4 p4[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      f32x4 acc = zero4();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) acc = M::mma(frag_along_row_swz<DK>(k_s, 16 * st, 4 * ks, lane), qf[ks], acc);
      const f32x4 cs = *reinterpret_cast<const f32x4*>(&S.cl[16 * st + 4 * g]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float y = acc[r] * fast_exp2(ct - cs[r]);
        acc[r] = 16 * st + 4 * g + r <= t_own ? y : 0.f;
      }
      p4[st] = pack(acc);
    }
    pg[0] = join(p4[0], p4[1]);
    pg[1] = join(p4[2], p4[3]);
  }
  // ---- W^T = (K gamma)^T T_G^T and U^T = V^T T_G^T (columns t): W to LDS, both kept
  bf16x4 wreg[KT];
  f32x4 ureg[VT];
  {
    frag zf[2], zg[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      zf[ks] = frag_along_row_perm<C>(z_s, 16 * w, 32 * ks, lane);
      const f32x4 g0 = *reinterpret_cast<const f32x4*>(&S.gm[32 * ks + 4 * g]);
      const f32x4 g1 = *reinterpret_cast<const f32x4*>(&S.gm[32 * ks + 16 + 4 * g]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        zg[ks][r] = static_cast<bf>(static_cast<float>(zf[ks][r]) * g0[r]);
        zg[ks][4 + r] = static_cast<bf>(static_cast<float>(zf[ks][4 + r]) * g1[r]);
      }
    }
    if (w < 2) zf[1] = zg[1] = frag{};  // above the diagonal (not formed)
#pragma unroll
    for (int mt = 0; mt < KT; ++mt) {
      f32x4 acc = M::mma(frag_down_rows_swz<DK>(k_s, 0, 16 * mt, lane), zg[0], zero4());
      acc = M::mma(frag_down_rows_swz<DK>(k_s, 32, 16 * mt, lane), zg[1], acc);
      wreg[mt] = pack(acc);
      *reinterpret_cast<bf16x4*>(S.w + swz<DK>(t_own, 2 * mt + (g >> 1)) + 4 * (g & 1)) = wreg[mt];
    }
#pragma unroll
    for (int mt = 0; mt < VT; ++mt) {
      ureg[mt] = M::mma(frag_down_rows_swz<DV>(S.v, 0, 16 * mt, lane), zf[0], zero4());
      ureg[mt] = M::mma(frag_down_rows_swz<DV>(S.v, 32, 16 * mt, lane), zf[1], ureg[mt]);
    }
  }
  // ONE: the output transposed, so that a lane holds four columns of its row
  auto out_mma = [](frag a, frag b, f32x4 c) { return ONE ? M::mma(b, a, c) : M::mma(a, b, c); };
  // ---- A_c^T = T_G^T P_G^T, masked by the levels of the chunk; intra-chunk output rows t
  f32x4 oacc[VT];
  {
    bf16x4 a4[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      f32x4 acc = zero4();
#pragma unroll
      for (int ks = st / 2; ks < 2; ++ks) acc = M::mma(frag_down_rows_swz<C>(z_s, 32 * ks, 16 * st, lane), pg[ks], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 16 * st + 4 * g + r;
        float x = acc[r];
        if constexpr (HAS_LAMBDA) x *= lam_h[t_own * NL + level_local(t_own, s)];
        acc[r] = s <= t_own ? x : 0.f;
      }
      a4[st] = pack(acc);
    }
    const frag a0 = join(a4[0], a4[1]), a1 = join(a4[2], a4[3]);
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) {
      oacc[vt] = out_mma(a0, frag_down_rows_swz<DV>(S.v, 0, 16 * vt, lane), zero4());
      oacc[vt] = out_mma(a1, frag_down_rows_swz<DV>(S.v, 32, 16 * vt, lane), oacc[vt]);
    }
  }
  __syncthreads();  // W of both chunks

  // ---- Qc^T = gamma Q^T - W^T P_G^T (columns t); U over the wave's own rows of Q
  f32x4 qc[KT];
  if (!ONE || (hf == 1 && N > 1)) {
    const float gt = S.gm[t_own];
#pragma unroll
    for (int mt = 0; mt < KT; ++mt) {
      const bf16x4 qv = *reinterpret_cast<const bf16x4*>(S.q + swz<DK>(t_own, 2 * mt + (g >> 1)) + 4 * (g & 1));
      f32x4 acc = M::mma(frag_down_rows_swz<DK>(S.w, 0, 16 * mt, lane), pg[0], zero4());
      acc = M::mma(frag_down_rows_swz<DK>(S.w, 32, 16 * mt, lane), pg[1], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) qc[mt][r] = gt * static_cast<float>(qv[r]) - acc[r];
    }
  }
  // Qc pieces: tiles mt, mt + 1 at once (pair_rows)
  bf* qc_row = qc_out + cidx * (C * DK) + t_own * DK + 16 * (g & 1) + 8 * (g >> 1);
  float* oin = oin_out + cidx * (C * DV) + w * (VT * 256) + 4 * lane;
  // U of chunk 1 in fp32, handed to the wave of chunk 0 that continues it, over V (no longer read)
  float* u1 = reinterpret_cast<float*>(w < 2 ? S1.v : S0.v) + (w & 1) * (VT * 256) + 4 * lane;
  bf* o_row = o_out + ((cur.tok0 + t_own) * H + cur.h) * DV + 16 * (g & 1) + 8 * (g >> 1);
  auto store_out = [&]() {  // rows of the output, as those of Qc
#pragma unroll
    for (int vt = 0; vt < VT; vt += 2)
      *reinterpret_cast<bf16x8*>(o_row + 16 * vt) = pair_rows(pack(oacc[vt]), pack(oacc[vt + 1]));
  };
  if (hf == 0) {
#pragma unroll
    for (int mt = 0; mt < VT; ++mt)
      *reinterpret_cast<bf16x4*>(S.q + swz<DV>(t_own, 2 * mt + (g >> 1)) + 4 * (g & 1)) = pack(ureg[mt]);
    if constexpr (ONE) {
      if (valid) store_out();
    } else {
#pragma unroll
      for (int mt = 0; mt < KT; mt += 2)
        *reinterpret_cast<bf16x8*>(qc_row + 16 * mt) = pair_rows(pack(qc[mt]), pack(qc[mt + 1]));
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) *reinterpret_cast<f32x4*>(oin + 256 * vt) = oacc[vt];
    }
  } else if constexpr (!ONE) {
#pragma unroll
    for (int mt = 0; mt < VT; ++mt) *reinterpret_cast<f32x4*>(u1 + 256 * mt) = ureg[mt];
  }
  __syncthreads();  // U of both chunks

  // ---- chunk 1 through chunk 0: half 1 its queries and output, half 0 its W and U (wave w: row tile w)
  const float g0 = S0.gm[C - 1];
  // x (rows of chunk 1, operand fragments over d) times K~_0^T, transposed (k = s of chunk 0)
  auto through = [&](const frag (&x)[KS], f32x4 (&out)[4]) {
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      f32x4 acc = zero4();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) acc = M::mma(frag_along_row_perm<DK>(S0.k, 16 * st, 32 * ks, lane), x[ks], acc);
      out[st] = acc * *reinterpret_cast<const f32x4*>(&S0.dc[16 * st + 4 * g]);
    }
  };
  if (hf == 1 && (!ONE || N > 1)) {
    const float l7 = HAS_LAMBDA ? lam_h[t_own * NL + NL - 1] : 1.f;
    frag gq[2], gl[2];  // the second times lambda
    {
      frag qf[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) qf[ks] = join(pack(qc[2 * ks]), pack(qc[2 * ks + 1]));
      f32x4 aq[4];
      through(qf, aq);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        gq[ks] = join(pack(aq[2 * ks]), pack(aq[2 * ks + 1]));
        gl[ks] = join(pack(aq[2 * ks] * l7), pack(aq[2 * ks + 1] * l7));
      }
    }
    if constexpr (!ONE) {
#pragma unroll
      for (int mt = 0; mt < KT; ++mt) {
        f32x4 x = M::mma(frag_down_rows_swz<DK>(S0.w, 0, 16 * mt, lane), gq[0], zero4());
        x = M::mma(frag_down_rows_swz<DK>(S0.w, 32, 16 * mt, lane), gq[1], x);
#pragma unroll
        for (int r = 0; r < 4; ++r) qc[mt][r] = g0 * qc[mt][r] - x[r];
      }
    }
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) {
      oacc[vt] = out_mma(gl[0], frag_down_rows_swz<DV>(S0.q, 0, 16 * vt, lane), oacc[vt]);
      oacc[vt] = out_mma(gl[1], frag_down_rows_swz<DV>(S0.q, 32, 16 * vt, lane), oacc[vt]);
    }
    if (!ONE && valid) {
#pragma unroll
      for (int mt = 0; mt < KT; mt += 2)
        *reinterpret_cast<bf16x8*>(qc_row + 16 * mt) = pair_rows(pack(qc[mt]), pack(qc[mt + 1]));
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) *reinterpret_cast<f32x4*>(oin + 256 * vt) = oacc[vt];
    }
  } else if (!ONE) {
    auto w_at = [&](int mt) { return reinterpret_cast<bf16x4*>(S1.w + swz<DK>(t_own, 2 * mt + (g >> 1)) + 4 * (g & 1)); };
    frag wf[KS], gw[2];
    f32x4 aw[4];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) wf[ks] = join(*w_at(2 * ks), *w_at(2 * ks + 1));
    through(wf, aw);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) gw[ks] = join(pack(aw[2 * ks]), pack(aw[2 * ks + 1]));
#pragma unroll
    for (int mt = 0; mt < KT; ++mt) {
      f32x4 x = M::mma(frag_down_rows_swz<DK>(S0.w, 0, 16 * mt, lane), gw[0], zero4());
      x = M::mma(frag_down_rows_swz<DK>(S0.w, 32, 16 * mt, lane), gw[1], x);
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = g0 * static_cast<float>(wf[mt / 2][4 * (mt & 1) + r]) - x[r];
      *w_at(mt) = pack(x);
    }
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) {
      f32x4 x = M::mma(frag_down_rows_swz<DV>(S0.q, 0, 16 * vt, lane), gw[0], zero4());
      x = M::mma(frag_down_rows_swz<DV>(S0.q, 32, 16 * vt, lane), gw[1], x);
      const f32x4 u = *reinterpret_cast<const f32x4*>(u1 + 256 * vt);
      *reinterpret_cast<bf16x4*>(S1.q + swz<DV>(t_own, 2 * vt + (g >> 1)) + 4 * (g & 1)) = pack(u - x);
    }
  }
  if constexpr (ONE) {
    if (hf == 1 && valid) store_out();
  } else {
    __syncthreads();  // W_1', U_1'
  }

  // ---- P = gamma_0 gamma_1 I - K~^T W (half 0) and H = K~^T U (half 1) over the pair's 128 tokens: RT row
  //      tiles of d_k per wave, their K~ fragments scaled once, each operand of W or U read for all of them
  constexpr int RT = KT / 4;
  const float gt1 = S1.gm[C - 1], gp = g0 * gt1;
  frag ka[RT][4];
  if constexpr (!ONE)
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const PairHalf<DK, DV>& X = half_s[ks >> 1];
    const int r0 = 32 * (ks & 1);
    const float sc = ks < 2 ? gt1 : 1.f;
    const f32x4 d0 = *reinterpret_cast<const f32x4*>(&X.dc[r0 + 4 * g]) * sc;
    const f32x4 d1 = *reinterpret_cast<const f32x4*>(&X.dc[r0 + 16 + 4 * g]) * sc;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      ka[i][ks] = frag_down_rows_swz<DK>(X.k, r0, 16 * (RT * w + i), lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ka[i][ks][r] = static_cast<bf>(static_cast<float>(ka[i][ks][r]) * d0[r]);
        ka[i][ks][4 + r] = static_cast<bf>(static_cast<float>(ka[i][ks][4 + r]) * d1[r]);
      }
    }
  }
  if (it + gridDim.x < npairs) {
    cur = where(it + gridDim.x);
    load_inputs(cur, tid);
  } else {  // no value of this turn is kept to the next (the registers are free in between)
    la_r = bt_r = 0.f;
#pragma unroll
    for (int e = 0; e < NLW; ++e) lam_r[e] = 0.f;
#pragma unroll
    for (int e = 0; e < PCS; ++e) kpre[e] = qpre[e] = vpre[e] = bf16x8{};
  }
  // product tiles (column tiles nt, nt + 1 of W or U), in the kfrag layout (eight rows of a column per
  // lane) or row-major from the transposed product (eight columns of a row)
  auto products = [&](auto is_p, auto transposed, bf* out) {
    constexpr bool P = decltype(is_p)::value, TR = decltype(transposed)::value;
#pragma unroll 1
    for (int nt = 0; nt < KT; nt += 2) {
      f32x4 acc[2][RT];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < RT; ++i) acc[c][i] = zero4();
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const frag x = frag_down_rows_swz<DK>(P ? half_s[ks >> 1].w : half_s[ks >> 1].q, 32 * (ks & 1), 16 * (nt + c), lane);
#pragma unroll
          for (int i = 0; i < RT; ++i) acc[c][i] = TR ? M::mma(x, ka[i][ks], acc[c][i]) : M::mma(ka[i][ks], x, acc[c][i]);
        }
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        const int rt = RT * w + i;
        if constexpr (P) {
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const int d = 16 * rt + (TR ? r16 : 4 * g), e = 16 * (nt + c) + (TR ? 4 * g : r16);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[c][i][r] = ((TR ? d == e + r : d + r == e) ? gp : 0.f) - acc[c][i][r];
          }
        }
        const int n8 = 8 * (g >> 1), n = nt + (g & 1);  // the lane's piece: rows (or columns) n8 .. + 7 of tile n
        *reinterpret_cast<bf16x8*>(out + (TR ? (16 * rt + r16) * DK + 16 * n + n8 : kfrag_idx<DK>(16 * rt + n8, 16 * n + r16))) =
            pair_rows(pack(acc[0][i]), pack(acc[1][i]));
      }
    }
  };
  if constexpr (ONE) continue;
  bf* pz = pz_out + (bh * N2 + zp) * (DK * DK);
  bf* hz = hz_out + (bh * N2 + zp) * (DK * DV);
  if (hf == 1) products(std::false_type{}, std::false_type{}, hz);
  else if (zp & 1) products(std::true_type{}, std::true_type{}, pz);
  else products(std::true_type{}, std::false_type{}, pz);
  }  // pair loop
}

// ---------------------------------------------------------------------------------------------
// Kernel 2: one level m >= 1 of the block tree.  Block (m, k) of a sequence covers pairs of chunks
// [k 2^m, (k + 1) 2^m).  It is formed from blocks lo = 2k and hi = 2k + 1 of level m - 1:
// T = T_hi T_lo, A = T_hi A_lo + A_hi, fp32 accumulation, one RNE cast.  Storage of a block:
// T (DK x DK) then A (DK x DV), A in the kfrag layout, T in the kfrag layout when k is even (the
// source groups that chunks read, and the lo side of the next level) and row-major when k is odd
// (the hi side).  Level 0 is the pair kernel's P and H (same layout rule, by pair parity).
// The (DK + DV) / 16 column tiles of [T | A] are split over workgroups of kCombineTiles column
// tiles, which the dispatch-order remap keeps on one XCD; wave w forms rows 16 (RT w + i) + 0..15
// of its workgroup's tiles (RT = DK / 64).  An odd block's T is formed transposed
// (T^T = T_lo^T T_hi^T) so that its rows are stored whole.  Every operand fragment of a workgroup
// is loaded up front; the B-operand fragments, the same for every wave, go through LDS.
// ---------------------------------------------------------------------------------------------
constexpr int kCombineTiles = 4;  // column tiles per workgroup

template <int DK, int DV>
__global__ __launch_bounds__(256) void k_gdn_combine(const bf* __restrict__ t_in, const bf* __restrict__ a_in,
                                                     int64_t t_stride, int64_t a_stride, int64_t n_in,
                                                     bf* __restrict__ out, int64_t n_out) {
  using MF = Mfma<bf>;
  typedef MF::frag frag;
  constexpr int KS = DK / 32, RT = DK / 64;  // k steps; row tiles per wave
  constexpr int TT = DK / 16, AT = DV / 16;  // column tiles of T and A
  constexpr int CT = kCombineTiles, S = (TT + AT) / CT;
  static_assert(TT % CT == 0 && AT % CT == 0, "a workgroup's tiles lie in T or in A");
  static_assert(CT * KS % 4 == 0, "the B fragments split evenly over the four waves");
  constexpr int BS = DK * (DK + DV);
  const int64_t id = xcd_remap(blockIdx.x, (int64_t)gridDim.x);
  const int64_t kb = id / S, bh = blockIdx.y;
  const int c0 = (int)(id % S) * CT;  // first column tile of [T | A]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, g = lane >> 4;
  const bf* tlo = t_in + (bh * n_in + 2 * kb) * t_stride;
  const bf* thi = tlo + t_stride;
  const bf* alo = a_in + (bh * n_in + 2 * kb) * a_stride;
  const bf* ahi = alo + a_stride;
  bf* tout = out + (bh * n_out + kb) * BS;
  bf* aout = tout + DK * DK;
  const bool t_part = c0 < TT, transposed = t_part && (kb & 1);

  // A operand: rows of T_hi (row-major), or for a transposed T the rows of T_lo^T (kfrag of T_lo);
  // rows 16 (RT wave + i) + r16, k = 32 ks + 8 g + 0..7
  frag fa[RT][KS];
  // B operand of column tile c0 + c: A_lo or T_lo (kfrag), or for a transposed T the rows of T_hi.
  // The same for every wave: each wave loads a quarter of them into LDS and reads all back.
  __shared__ frag fb_s[CT * KS][64];
  constexpr int FPW = CT * KS / 4;  // B fragments loaded per wave
  frag fbw[FPW];
#pragma unroll
  for (int x = 0; x < FPW; ++x) {
    const int f = wave + 4 * x, c = f / KS, ks = f % KS;
    const int nt = t_part ? c0 + c : c0 - TT + c;
    fbw[x] = transposed ? MF::load(thi + (16 * nt + r16) * DK + 32 * ks + 8 * g)
                        : MF::load((t_part ? tlo : alo) + ((nt * KS + ks) * 64 + lane) * 8);
  }
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      fa[i][ks] = transposed ? MF::load(tlo + (((RT * wave + i) * KS + ks) * 64 + lane) * 8)
                             : MF::load(thi + (16 * (RT * wave + i) + r16) * DK + 32 * ks + 8 * g);
  // A_hi (added to the A tiles) with the operands, not after the products
  bf16x4 ahv[CT][RT];
  if (!t_part) {
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int i = 0; i < RT; ++i)
        ahv[c][i] = *reinterpret_cast<const bf16x4*>(ahi + kfrag_idx<DK>(16 * (RT * wave + i) + 4 * g, 16 * (c0 - TT + c) + r16));
  }
#pragma unroll
  for (int x = 0; x < FPW; ++x) fb_s[wave + 4 * x][lane] = fbw[x];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int nt = t_part ? c0 + c : c0 - TT + c;
    f32x4 acc[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int i = 0; i < RT; ++i) acc[i] = MF::mma(fa[i][ks], fb_s[c * KS + ks][lane], acc[i]);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int row0 = 16 * (RT * wave + i) + 4 * g;
      bf16x4 res;
      if (!t_part) {  // A = T_hi A_lo + A_hi; the lane's four rows are four consecutive kfrag elements
        const int idx = kfrag_idx<DK>(row0, 16 * nt + r16);
        const bf16x4 add = ahv[c][i];
#pragma unroll
        for (int r = 0; r < 4; ++r) res[r] = static_cast<bf>(acc[i][r] + static_cast<float>(add[r]));
        *reinterpret_cast<bf16x4*>(aout + idx) = res;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) res[r] = static_cast<bf>(acc[i][r]);
        if (!transposed)  // T = T_hi T_lo, kfrag
          *reinterpret_cast<bf16x4*>(tout + kfrag_idx<DK>(row0, 16 * nt + r16)) = res;
        else  // lane value r is T[16 nt + r16][row0 + r]: row-major T
          *reinterpret_cast<bf16x4*>(tout + (16 * nt + r16) * DK + row0) = res;
      }
    }
  }
}

// Element offset of tree level m >= 1 in the tree region (levels 1 .. m-1 before it).
__device__ __host__ inline int64_t tree_level_offset(int64_t BH, int64_t N, int m, int64_t block_size) {
  int64_t off = 0;
  for (int x = 1; x < m; ++x) off += BH * (N >> x) * block_size;
  return off;
}

// ---------------------------------------------------------------------------------------------
// Kernel 3: read-out.  One workgroup (4 waves) per chunk z.  The chunk's Q~ rows (already through its
// pair's first chunk) are carried through its source groups from the lowest set bit of z >> 1 up: at level
// j >= 2 (bit j - 1 of z set) the rows add lambda_t^(log2 C + j) q~_t^T A(G_j) and, if a higher bit follows,
// become q~^T T(G_j).  The
// node fragments come straight from global memory in the kfrag layout; Q~ lives in LDS (double
// buffered, bf16); wave w owns the output columns DV/4 w .. and the Q~ columns DK/4 w .. .  The
// chunk's intra-chunk output is added at the end and the rows are stored through LDS.
// lambda == NULL: every level weight is 1 (Gated DeltaNet: the whole prefix state).
// Bound: one node round trip per level, 3 levels per chunk at T = 8192.  8 waves per pair of chunks, each node
// read once for both, one column tile per wave: tree and read-out 216 -> 264 us at T = 8192, d = 128 (two
// workgroups per compute unit with half the loads in flight, and spills).
// ---------------------------------------------------------------------------------------------
template <int C, int DK, int DV, bool HAS_LAMBDA>
__global__ __launch_bounds__(256, 2) void k_gdn_read(const float* __restrict__ lam, const bf* __restrict__ qc_in,
                                                  const bf* __restrict__ pz, const bf* __restrict__ hz,
                                                  const bf* __restrict__ tree, const float* __restrict__ oin_in,
                                                  bf* __restrict__ o, int64_t Tlen, int H, int L, int BH) {
  using MF = Mfma<bf>;
  typedef MF::frag frag;
  constexpr int LOG2C = (C == 16) ? 4 : (C == 32) ? 5 : 6;
  constexpr int KS = DK / 32, RT = C / 16;  // k steps; row tiles (all of them, every wave)
  constexpr int VT = DV / 64, KT = DK / 64; // column tiles of this wave: output, carried Q~
  constexpr int LDQ = DK + 8;
  constexpr int BS = DK * (DK + DV);
  static_assert(C == 64 && VT >= 1 && KT >= 1, "four row tiles, whole column tiles per wave");
  static_assert(2 * C * LDQ * 2 >= C * DV * 4, "the output staging fits the Q~ buffers");
  __shared__ __attribute__((aligned(16))) bf q_s[2][C * LDQ];
  __shared__ float lw_s[HAS_LAMBDA ? C * kMaxJ : 1];

  const int64_t N = Tlen / C;
  const int64_t work = xcd_remap(blockIdx.x, (int64_t)gridDim.x);  // (b h, z): a sequence's chunks on one XCD
  const int64_t z = work % N, bh = work / N;
  const int h = (int)(bh % H), b = (int)(bh / H);
  const int64_t cidx = bh * N + z;
  const int64_t tok0 = (int64_t)b * Tlen + z * C;
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t zp = z >> 1, N2 = (N + 1) >> 1;  // the chunk's pair; pairs of the sequence
  const int J = N2 <= 1 ? 0 : 32 - __builtin_clz((unsigned)(N2 - 1));

  // node fragments of the level at bit m: A(G) for this wave's output columns, and T(G) for its
  // q~ columns when a higher level follows.  The first level's are loaded before Q~ is staged.
  frag ba[VT][KS], bt[KT][KS];
  auto load_level = [&](int m, bool with_t) {
    const int64_t kblk = (zp >> m) - 1;
    const bf *tn, *an;
    if (m == 0) {
      tn = pz + (bh * N2 + kblk) * (DK * DK);
      an = hz + (bh * N2 + kblk) * (DK * DV);
    } else {
      tn = tree + tree_level_offset(BH, N2, m, BS) + (bh * (N2 >> m) + kblk) * BS;
      an = tn + DK * DK;
    }
#pragma unroll
    for (int v = 0; v < VT; ++v)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) ba[v][ks] = MF::load(an + (((VT * wave + v) * KS + ks) * 64 + lane) * 8);
    if (with_t) {
#pragma unroll
      for (int v = 0; v < KT; ++v)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) bt[v][ks] = MF::load(tn + (((KT * wave + v) * KS + ks) * 64 + lane) * 8);
    }
  };
  unsigned bits = (unsigned)zp;
  if (bits) load_level(__builtin_ctz(bits), (bits & (bits - 1)) != 0);

  for (int x = tid; x < C * DK / 8; x += 256) {
    const int t = x / (DK / 8), c = x % (DK / 8);
    *reinterpret_cast<bf16x8*>(&q_s[0][t * LDQ + 8 * c]) =
        *reinterpret_cast<const bf16x8*>(qc_in + cidx * (C * DK) + t * DK + 8 * c);
  }
  if constexpr (HAS_LAMBDA) {
    for (int x = tid; x < C * J; x += 256) {
      const int t = x / J, jj = x % J;
      lw_s[t * kMaxJ + jj] = lam[((tok0 + t) * H + h) * L + LOG2C + 2 + jj];
    }
  }
  __syncthreads();

  f32x4 acc[RT][VT];
#pragma unroll
  for (int mt = 0; mt < RT; ++mt)
#pragma unroll
    for (int v = 0; v < VT; ++v) acc[mt][v] = f32x4{0.f, 0.f, 0.f, 0.f};
  int cur = 0;
  bool first = true;
  while (bits) {
    const int m = __builtin_ctz(bits);  // tree level of the source group; token level log2 C + m + 2
    bits &= bits - 1;
    if (!first) load_level(m, bits != 0);
    first = false;
    // q~ A(G) for this wave's output columns and, when a higher level follows, q~ T(G) for its
    // q~ columns, from one read of each q~ fragment
    const bf* qs = q_s[cur];
    f32x4 part[RT][VT], qn[RT][KT];
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) {
#pragma unroll
      for (int v = 0; v < VT; ++v) part[mt][v] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < KT; ++v) qn[mt][v] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int mt = 0; mt < RT; ++mt) {
        const frag a = *reinterpret_cast<const bf16x8*>(&qs[(16 * mt + r16) * LDQ + 32 * ks + 8 * g]);
#pragma unroll
        for (int v = 0; v < VT; ++v) part[mt][v] = MF::mma(a, ba[v][ks], part[mt][v]);
        if (bits) {
#pragma unroll
          for (int v = 0; v < KT; ++v) qn[mt][v] = MF::mma(a, bt[v][ks], qn[mt][v]);
        }
      }
#pragma unroll
    for (int mt = 0; mt < RT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float w = HAS_LAMBDA ? lw_s[(16 * mt + 4 * g + r) * kMaxJ + m] : 1.f;
#pragma unroll
        for (int v = 0; v < VT; ++v) acc[mt][v][r] += w * part[mt][v][r];
      }
    if (bits) {
      bf* qd = q_s[cur ^ 1];
#pragma unroll
      for (int mt = 0; mt < RT; ++mt)
#pragma unroll
        for (int v = 0; v < KT; ++v)
#pragma unroll
          for (int r = 0; r < 4; ++r) qd[(16 * mt + 4 * g + r) * LDQ + 16 * (KT * wave + v) + r16] = static_cast<bf>(qn[mt][v][r]);
      __syncthreads();  // the carried rows complete; every wave is done with the old ones
      cur ^= 1;
    }
  }

  // o = intra-chunk output (stored by the chunk kernel in this accumulator layout) + the levels,
  // rows staged through LDS (over the Q~ buffers)
  const float* oin = oin_in + cidx * (C * DV);
  f32x4 oi[RT][VT];
#pragma unroll
  for (int mt = 0; mt < RT; ++mt)
#pragma unroll
    for (int v = 0; v < VT; ++v)
      oi[mt][v] = *reinterpret_cast<const f32x4*>(oin + ((mt * (DV / 16) + VT * wave + v) * 64 + lane) * 4);
  __syncthreads();
  float* o_s = reinterpret_cast<float*>(&q_s[0][0]);
#pragma unroll
  for (int mt = 0; mt < RT; ++mt)
#pragma unroll
    for (int v = 0; v < VT; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        o_s[(16 * mt + 4 * g + r) * DV + 16 * (VT * wave + v) + r16] = oi[mt][v][r] + acc[mt][v][r];
  __syncthreads();
  for (int x = tid; x < C * DV / 8; x += 256) {
    const int t = x / (DV / 8), c = 8 * (x % (DV / 8));
    const f32x4 s0 = *reinterpret_cast<const f32x4*>(o_s + t * DV + c);
    const f32x4 s1 = *reinterpret_cast<const f32x4*>(o_s + t * DV + c + 4);
    bf16x8 res;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      res[e] = static_cast<bf>(s0[e]);
      res[4 + e] = static_cast<bf>(s1[e]);
    }
    *reinterpret_cast<bf16x8*>(o + ((tok0 + t) * H + h) * DV + c) = res;
  }
}

}  // namespace gdn

// ---------------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------------
int64_t gdn_workspace(int64_t B, int64_t T, int64_t H, int64_t dk, int64_t dv, int64_t C, GdnLayout* lay) {
  const int64_t N = T / C, BHN = B * H * N, N2 = (N + 1) / 2, BHP = B * H * N2;
  auto al = [](int64_t x) { return (x + 255) & ~int64_t(255); };
  GdnLayout w{};
  int64_t cur = 0;
  w.qc = cur; cur += al(BHN * C * dk * 2);
  w.pz = cur; cur += al(BHP * dk * dk * 2);
  w.hz = cur; cur += al(BHP * dk * dv * 2);
  w.oin = cur; cur += al(BHN * C * dv * 4);
  int64_t blocks = 0;  // tree levels 1 .. J-1 (the source groups of 2 .. 2^(J-1) pairs of chunks)
  for (int64_t m = 1; (int64_t(1) << m) < N2; ++m) blocks += N2 >> m;
  w.tree = cur; cur += al(B * H * blocks * dk * (dk + dv) * 2);
  w.total = cur;
  if (lay) *lay = w;
  return cur;
}

// Enqueues the two stages on `st`.  With `ev` non-null, ev[0] is recorded before the chunk
// kernel, ev[1] after it and ev[2] after the tree and read-out kernels (used by the staged entry
// point).
template <int C, int DK, int DV>
hipError_t launch_gdn(const GdnArgs& a, hipStream_t st, hipEvent_t* ev) {
  GdnLayout w;
  gdn_workspace(a.B, a.T, a.H, DK, DV, C, &w);
  char* base = static_cast<char*>(a.workspace);
  __bf16* qc = reinterpret_cast<__bf16*>(base + w.qc);
  __bf16* pz = reinterpret_cast<__bf16*>(base + w.pz);
  __bf16* hz = reinterpret_cast<__bf16*>(base + w.hz);
  float* oin = reinterpret_cast<float*>(base + w.oin);
  const int64_t N = a.T / C, N2 = (N + 1) / 2;
  const int J = N2 <= 1 ? 0 : 64 - __builtin_clzll(uint64_t(N2 - 1));
  const int64_t nchunks = a.B * a.H * N;
  // the pair kernel runs one persistent workgroup per compute unit
  const int64_t npairs = N == 1 ? (a.B * a.H + 1) / 2 : a.B * a.H * N2;
  int dev = 0, ncu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
    ncu = 256;
  const dim3 g1((unsigned)(npairs < ncu ? npairs : ncu));
  const __bf16* q = static_cast<const __bf16*>(a.q);
  const __bf16* k = static_cast<const __bf16*>(a.k);
  const __bf16* v = static_cast<const __bf16*>(a.v);
  __bf16* o = static_cast<__bf16*>(a.o);
  if (ev) (void)hipEventRecord(ev[0], st);
  auto launch_pair = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, g1, dim3(512), 0, st, q, k, v, a.log_alpha, a.beta, a.lambda, qc, pz, hz, oin, o, a.T,
                       (int)a.H, a.L, npairs, a.B * a.H);
  };
  const bool one = N2 == 1;  // no tree, nothing to read out
  if (a.lambda && one) launch_pair(gdn::k_gdn_pair<DK, DV, true, true>);
  else if (a.lambda) launch_pair(gdn::k_gdn_pair<DK, DV, true, false>);
  else if (one) launch_pair(gdn::k_gdn_pair<DK, DV, false, true>);
  else launch_pair(gdn::k_gdn_pair<DK, DV, false, false>);
  if (ev) (void)hipEventRecord(ev[1], st);
  // the block tree, one level per launch (level m from level m - 1; level 0 = P_z, H_z)
  __bf16* tree = reinterpret_cast<__bf16*>(base + w.tree);
  const int64_t BH = a.B * a.H, BS = (int64_t)DK * (DK + DV);
  for (int m = 1; m < J; ++m) {
    const __bf16* tin = m == 1 ? pz : tree + gdn::tree_level_offset(BH, N2, m - 1, BS);
    const __bf16* ain = m == 1 ? hz : tin + DK * DK;
    const int64_t ts = m == 1 ? DK * DK : BS, as = m == 1 ? DK * DV : BS;
    const int64_t nin = m == 1 ? N2 : (N2 >> (m - 1));
    constexpr int split = (DK + DV) / 16 / gdn::kCombineTiles;
    hipLaunchKernelGGL((gdn::k_gdn_combine<DK, DV>), dim3((unsigned)((N2 >> m) * split), (unsigned)BH), dim3(256), 0, st,
                       tin, ain, ts, as, nin, tree + gdn::tree_level_offset(BH, N2, m, BS), N2 >> m);
  }
  auto launch_read = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)nchunks), dim3(256), 0, st, a.lambda, qc, pz, hz, tree, oin, o, a.T,
                       (int)a.H, a.L, (int)BH);
  };
  if (!one && a.lambda) launch_read(gdn::k_gdn_read<C, DK, DV, true>);
  else if (!one) launch_read(gdn::k_gdn_read<C, DK, DV, false>);
  if (ev) (void)hipEventRecord(ev[2], st);
  return hipGetLastError();
}

#define LL_GDN_SHAPES(X) \
  X(64, 64, 64)          \
  X(64, 128, 128)

const GdnEntry* gdn_table(int* n) {
#define LL_ENTRY(C, DK, DV) {C, DK, DV, &launch_gdn<C, DK, DV>},
  static const GdnEntry table[] = {LL_GDN_SHAPES(LL_ENTRY)};
#undef LL_ENTRY
  *n = sizeof(table) / sizeof(table[0]);
  return table;
}

}  // namespace ll
