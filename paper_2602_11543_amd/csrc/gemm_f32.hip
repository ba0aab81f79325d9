// Grouped fp32 GEMM on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 products and sums, no narrower type anywhere).
//
// Four wavefronts, each a 32 x 32 sub-tile as 2 x 2 MFMA tiles, over 32 k of a K-tile.  Spatially they form a BM x BN
// tile; where that leaves wavefronts over (WK > 1), the others take further 32-wide slices of k and the partial sums meet in
// LDS at the end, in a fixed order: the layers this path serves have a few hundred rows, and a block's serial K loop is what
// they wait for.  What bounds them is latency: launch, tile table, first loads, a handful of K-tiles.
// Operands come straight into LDS (lds_load.h), NS - 1 K-tiles ahead, in panels of 32 k: [row][32 k] for an operand whose
// contraction index is the fast axis (128-byte rows, chunks permuted as in gemm_mfma.hip), [32 k][row] otherwise.  One
// 16-byte LDS read of the first kind is four MFMAs' worth of one fragment, and one 8-byte read of the second kind one
// MFMA's worth of two; for that the MFMAs take the k of a slice in the order 16 (s/4) + 4 q + s%4 (MFMA s, lane group
// q), and a K-strided operand's fragment i holds the rows 2 l + i.
// Sums run in two levels, 128 terms and then their totals, so rounding grows with sqrt(128) + sqrt(K / 128).
// Against the vector-ALU kernel (gemm_simt.hip: guarded four-byte loads, one K-tile in flight), us: 512 tokens 256 x 512, 8
// experts, top-2: gate + up 56 -> 16, down 35 -> 9.5, its dgrad 35 -> 15, dgrad gate + up 65 -> 16, weight gradients 29 -> 13, the step
// 269 -> 90.  Steps of 2000 tokens 768 x 1024, 16 experts, top-8: 5039 -> 1604 (94 TFLOP/s of the 157 that the instruction
// has); 300 tokens 256 x 1000, 32 experts, top-8: 590 -> 223; 64 tokens 128 x 128, 64 experts: 129 -> 57.
#include <type_traits>

#include "gemm.h"
#include "lds_load.h"
#include "plan.h"

namespace spes {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;

template <int BM_, int BN_, int WK_, int NS_>
struct Cfg {
  static constexpr int BM = BM_, BN = BN_, WK = WK_, NS = NS_;     // WK: slices of k side by side, NS: K-tiles in LDS
  static constexpr int WN = BN / 32, BK = 32 * WK;
  static constexpr int NA = BM * WK / 32, NB = BN * WK / 32;       // 1 KB loads per wavefront and K-tile
  static constexpr int A_VEC = BM * WK * 8, STAGE_VEC = (BM + BN) * WK * 8;      // 16-byte units
  static_assert((BM / 32) * WN * WK == 4, "four wavefronts");
};

constexpr int kSetSlices = 4;      // slices of k of the weight gradients, on every tile

template <int MODE, int EPI, bool A_KC, bool B_KC, bool SETS, typename C>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(const GemmArgs g) {
  constexpr int BM = C::BM, BN = C::BN, BK = C::BK, WK = C::WK, NS = C::NS, NA = C::NA, NB = C::NB, NP = NA + NB;
  constexpr int BNO = EPI == kEpiSwiglu ? BN / 2 : BN;     // fused SwiGLU: 16 gate and 16 up columns per wavefront column
  __shared__ uint4 smem[NS * C::STAGE_VEC];
  const int tid = threadIdx.x, lane = tid & 63, wave = (int)uniform(tid >> 6);
  const int l16 = lane & 15, q = lane >> 4;
  const int wk = wave % WK, wm = wave / WK / C::WN, wn = wave / WK % C::WN;

  // ---- which tile ----
  const GemmArgs::Set st = g.set[SETS ? blockIdx.z % g.n_sets : 0];
  const int Mdim = SETS ? st.Mdim : g.Mdim, Ndim = SETS ? st.Ndim : g.Ndim;
  const long a_ks = SETS ? st.a_ks : g.a_ks, b_ks = SETS ? st.b_ks : g.b_ks, c_ms = SETS ? st.c_ms : g.c_ms;
  const bool a_gather = SETS && st.a_gather, b_gather = SETS && !a_gather;      // one of the two
  const int col_tiles = cdiv(Ndim, BNO);
  const int n0 = (MODE == kRaggedM ? blockIdx.x : blockIdx.x % col_tiles) * BNO;
  long m0, m_end, k_begin, k_end, b_group = 0, c_group = 0;
  bool store2 = true;
  if (MODE == kRaggedM) {
    if ((int)blockIdx.y >= *g.n_tiles) return;
    const int e = g.tile_expert[blockIdx.y];
    store2 = ((g.c2_skip >> e) & 1ull) == 0;
    m0 = g.tile_row0[blockIdx.y];
    m_end = min((long)g.offset[e + 1], m0 + BM);
    k_begin = 0; k_end = g.Kdim;
    b_group = (long)e * g.b_gs;
  } else {
    const int grp = SETS ? blockIdx.z / g.n_sets : blockIdx.z;
    m0 = (long)(blockIdx.x / col_tiles) * BM;
    if (m0 >= Mdim) return;
    m_end = min((long)Mdim, m0 + BM);
    if (g.offset != nullptr) {
      const int e = g.group_expert[grp];
      k_begin = g.offset[e]; k_end = g.offset[e + 1];
    } else {
      k_begin = (long)grp * g.kchunk; k_end = min((long)g.Kdim, k_begin + g.kchunk);
    }
    c_group = (long)grp * g.c_gs;
  }

  // ---- operands: buffer resources whose base moves with the K-tile; bytes from there to the operand's end (K-contiguous, gathered)
  // or to the end of the contraction range (K-strided), behind which loads deliver zeros ----
  const int klen = (int)uniform((unsigned)(k_end - k_begin));
  constexpr bool TWO_PASS = MODE == kRaggedM && EPI == kEpiStore && !B_KC;
  const int nk = klen > 0 ? (klen + BK - 1) / BK : 0, nsteps = TWO_PASS ? nk * g.npairs : nk;
  auto at = [](const void* p, long elems) -> unsigned long {
    const unsigned long v = reinterpret_cast<unsigned long>(p) + (unsigned long)(elems * 4);
    return (unsigned long)uniform((unsigned)(v >> 32)) << 32 | uniform((unsigned)v);
  };
  const long a_row0 = A_KC && !(MODE == kRaggedM && g.a_rows) ? m0 * g.a_ms : 0;      // a gathered operand is addressed from its start
  const long a_first = A_KC ? a_row0 + k_begin : a_gather ? 0 : k_begin * a_ks;
  const long b_first = b_group + (B_KC ? (long)n0 * g.b_ns + k_begin : b_gather ? 0 : k_begin * b_ks);
  const unsigned long a_base[2] = {at(SETS ? st.A : g.A[0], a_first), at(TWO_PASS ? g.A[1] : SETS ? st.A : g.A[0], a_first)};
  const unsigned long b_base[2] = {at(SETS ? st.B : g.B[0], b_first), at(TWO_PASS || EPI == kEpiSwiglu ? g.B[1] : SETS ? st.B : g.B[0], b_first)};
  auto left_bytes = [](long elems) { return (unsigned)min(elems * 4, 0xfffffff0L); };
  const unsigned a_step = uniform(A_KC ? 4u : a_gather ? 0u : (unsigned)(a_ks * 4)), b_step = uniform(B_KC ? 4u : b_gather ? 0u : (unsigned)(b_ks * 4));
  const unsigned a_bytes = uniform(A_KC || a_gather ? left_bytes((SETS ? st.a_elems : g.a_elems) - a_first) : (unsigned)klen * a_step);
  const unsigned b_bytes = uniform(B_KC || b_gather ? left_bytes((SETS ? st.b_elems : g.b_elems) - b_first) : (unsigned)klen * b_step);

  const int kc_chunk = (lane & 7) ^ ((wave * 4 + (lane >> 4)) & 7);
  constexpr int ACH = BM / 4, BCH = BN / 4, KRA = 256 / BM, KRB = 256 / BN;       // K-strided: 16-byte chunks per k-row, k-rows per load
  const int a_krow = wave * KRA + lane / ACH, b_krow = wave * KRB + lane / BCH;
  const unsigned a_col = (unsigned)((m0 + (lane % ACH) * 4) * 4), b_col = (unsigned)((n0 + (lane % BCH) * 4) * 4);
  auto clamped = [](unsigned long o) { return o < kOutOfRange ? (unsigned)o : kOutOfRange; };
  unsigned aoff[NA], boff[NB];
  int ak[NA], bk[NB];                  // k of a load's chunk within the K-tile (K-contiguous)
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    ak[i] = i * 32 / BM * 32 + kc_chunk * 4;
    if (A_KC) {
      const int row = i * 32 % BM + wave * 8 + (lane >> 3);
      long m = row;
      if (MODE == kRaggedM && g.a_rows) m = g.a_rows[m0 + row < m_end ? m0 + row : m_end - 1];
      aoff[i] = clamped((unsigned long)((m * g.a_ms + ak[i]) * 4));
    } else {
      aoff[i] = clamped((unsigned long)(a_krow + i * 4 * KRA) * (unsigned long)(a_ks * 4) + a_col);
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    bk[i] = i * 32 / BN * 32 + kc_chunk * 4;
    if (B_KC) {
      const int row = i * 32 % BN + wave * 8 + (lane >> 3);
      // fused SwiGLU: of every 32 tile rows 16 come from the gate matrix and 16 from the up matrix
      const long n = EPI == kEpiSwiglu ? row / 32 * 16 + row % 16 : row;
      boff[i] = clamped((unsigned long)((n * g.b_ns + bk[i]) * 4));
    } else {
      boff[i] = clamped((unsigned long)(b_krow + i * 4 * KRB) * (unsigned long)(b_ks * 4) + b_col);
    }
  }

  // k-rows of a K-tile from the index table (operand sets)
  int kidx[SETS ? NA : 1];
  static_assert(!SETS || (BM == BN && NA == NB), "one list of k-rows serves either operand");
  auto load_kidx = [&](int t) {
    if (SETS) {
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const int k = (int)k_begin + t * BK + a_krow + i * 4 * KRA;
        kidx[i] = g.k_rows[max(0, min(k, (int)k_end - 1))];
      }
    }
  };
  const unsigned lds0 = (unsigned)(unsigned long)(__attribute__((address_space(3))) uint4*)smem + (unsigned)wave * 1024u;
  auto load_tile = [&](int t, int slot) {
    const bool second = TWO_PASS && t >= nk;
    const int k0 = (t - (second ? nk : 0)) * BK, left = klen - k0;
    const bool live = t < nsteps;
    const unsigned ao = (unsigned)k0 * a_step, bo = (unsigned)k0 * b_step;
    const rsrc_t ra = make_rsrc(a_base[second ? 1 : 0] + ao, live ? a_bytes - ao : 0u);
    const rsrc_t rb = make_rsrc(b_base[second ? 1 : 0] + bo, live ? b_bytes - bo : 0u);
    const rsrc_t rb1 = make_rsrc(b_base[1] + bo, live ? b_bytes - bo : 0u);
    const unsigned dst = lds0 + (unsigned)slot * (C::STAGE_VEC * 16u);
    const unsigned g_pitch = (unsigned)((a_gather ? a_ks : b_ks) * 4), g_col = a_gather ? a_col : b_col;
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      unsigned off = aoff[i];
      if (A_KC) off = ak[i] < left ? off : kOutOfRange;
      if (SETS) {
        const unsigned go = a_krow + i * 4 * KRA < left ? (unsigned)kidx[i] * g_pitch + g_col : kOutOfRange;
        off = a_gather ? go : off;
      }
      const unsigned m0 = set_lds_dest(dst + (unsigned)i * 4096u);
      one_instruction();
      load_to_lds(ra, off, m0);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      unsigned off = boff[i];
      if (B_KC) off = bk[i] < left ? off : kOutOfRange;
      if (SETS) {
        const unsigned go = a_krow + i * 4 * KRA < left ? (unsigned)kidx[i] * g_pitch + g_col : kOutOfRange;
        off = a_gather ? off : go;
      }
      const unsigned m0 = set_lds_dest(dst + C::A_VEC * 16u + (unsigned)i * 4096u);
      one_instruction();
      if (EPI == kEpiSwiglu) {
        // a wavefront's eight tile rows are all gate rows or all up rows: rows 0-15 of every 32 are gate rows
        const bool up = (wave & 2) != 0;
        load_to_lds(rsrc_t{up ? rb1.x : rb.x, up ? rb1.y : rb.y, rb.z, rb.w}, off, m0);
      } else {
        load_to_lds(rb, off, m0);
      }
    }
  };

  // ---- main loop ----
  // KS sums side by side, K-tile t into sum t % KS.  Weight gradients: the slices of the tile that shares out k, so that the two tiles,
  // between which the number of trainable experts decides, add up in the same order.  (With one sum on the wide tile an
  // expert's gradients changed with the mask; the four cost a step of 1200 tokens 640 x 640 248 -> 255 us, of 2000 tokens 768 x 1024,
  // top-8, 1885 -> 1915, of 512 tokens 256 x 512 nothing.)
  constexpr int KS = SETS ? kSetSlices / WK : 1;
  f32x4 acc[KS][2][2], total[KS][2][2];        // [sum][column fragment][row fragment]
#pragma unroll
  for (int c = 0; c < KS; ++c)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < 2; ++i) { acc[c][j][i] = f32x4{0.f, 0.f, 0.f, 0.f}; total[c][j][i] = acc[c][j][i]; }
  const char* const lds = reinterpret_cast<const char*>(smem);
  for (int t = 0; t < NS - 1; ++t) {
    load_kidx(t);
    load_tile(t, t);
  }
  load_kidx(NS - 1);
  int slot = 0, fill = NS - 1;         // LDS slot of K-tile t and of the one to be loaded
  auto k_tile = [&](int t, auto sum) __attribute__((always_inline)) {
    constexpr int c = decltype(sum)::value;
    wait_and_meet<(NS - 2) * NP>();    // K-tile t is here, and K-tile t-1, whose slot is loaded now, has been read by all
    load_tile(t + NS - 1, fill);
    load_kidx(t + NS);
    const char* const sa = lds + slot * (C::STAGE_VEC * 16) + wk * (BM * 128);
    const char* const sb = lds + slot * (C::STAGE_VEC * 16) + C::A_VEC * 16 + wk * (BN * 128);
    float fa[2][8], fb[2][8];          // [fragment][MFMA]
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      const int pos = ((jj * 4 + q) ^ (l16 >> 1)) * 16;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (A_KC) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(sa + (wm * 32 + i * 16 + l16) * 128 + pos);
#pragma unroll
          for (int e = 0; e < 4; ++e) fa[i][jj * 4 + e] = v[e];
        }
        if (B_KC) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(sb + (wn * 32 + i * 16 + l16) * 128 + pos);
#pragma unroll
          for (int e = 0; e < 4; ++e) fb[i][jj * 4 + e] = v[e];
        }
      }
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int k = 16 * (s / 4) + 4 * q + s % 4;
      if (!A_KC) {
        const f32x2 v = *reinterpret_cast<const f32x2*>(sa + (k * BM + wm * 32 + 2 * l16) * 4);
        fa[0][s] = v[0]; fa[1][s] = v[1];
      }
      if (!B_KC) {
        const f32x2 v = *reinterpret_cast<const f32x2*>(sb + (k * BN + wn * 32 + 2 * l16) * 4);
        fb[0][s] = v[0]; fb[1][s] = v[1];
      }
    }
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[c][j][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][s], fa[i][s], acc[c][j][i], 0, 0, 0);
    if ((t / KS & 3) == 3) {           // 128 terms
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) { total[c][j][i] += acc[c][j][i]; acc[c][j][i] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    }
    slot = slot + 1 == NS ? 0 : slot + 1;
    fill = fill + 1 == NS ? 0 : fill + 1;
  };
  for (int t = 0; t < nsteps; t += KS) {
    k_tile(t, std::integral_constant<int, 0>{});
    if constexpr (KS > 1) {
      static_assert(KS == 4, "four sums");
      if (t + 1 < nsteps) k_tile(t + 1, std::integral_constant<int, 1>{});
      if (t + 2 < nsteps) k_tile(t + 2, std::integral_constant<int, 2>{});
      if (t + 3 < nsteps) k_tile(t + 3, std::integral_constant<int, 3>{});
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // no load may still write LDS: the sums use it, or the next block
  f32x4 result[2][2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      result[j][i] = total[0][j][i] + acc[0][j][i];
#pragma unroll
      for (int c = 1; c < KS; ++c) result[j][i] += total[c][j][i] + acc[c][j][i];
    }

  // ---- partial sums of the slices, added in order; wavefront wk of a sub-tile goes on with row fragment wk ----
  if (WK > 1) {
    f32x4* red = reinterpret_cast<f32x4*>(smem);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < 2; ++i) red[((wave * 2 + i) * 2 + j) * 64 + lane] = result[j][i];
    __syncthreads();
    if (wk >= 2) return;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      f32x4 sum = red[((((wave - wk) * 2) + wk) * 2 + j) * 64 + lane];
#pragma unroll
      for (int w = 1; w < WK; ++w) sum += red[(((wave - wk + w) * 2 + wk) * 2 + j) * 64 + lane];
      result[j][0] = sum;
    }
  }

  // ---- epilogue: a lane holds 4 (B K-contiguous: columns 16 j + 4 q + r) or 8 (K-strided: 8 q + 2 r + j) columns of one row per
  // row fragment ----
  const int nw = n0 + wn * (EPI == kEpiSwiglu ? 16 : 32);
  const bool vec = Ndim % 4 == 0 && c_ms % 4 == 0;     // (the router scores may have any number of columns)
#pragma unroll
  for (int u = 0; u < (WK > 1 ? 1 : 2); ++u) {
    const int i = WK > 1 ? wk : u;
    const long m = m0 + wm * 32 + (A_KC ? 16 * i + l16 : 2 * l16 + i);
    const bool m_in = m < m_end;
    const f32x4 v0 = result[0][u], v1 = result[1][u];
    if (EPI == kEpiSwiglu) {
      const int n = nw + 4 * q;
      if (m_in && n < Ndim) {
        const long ci = m * c_ms + n;
        f32x4 h;
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = v0[r] * sigmoidf_(v0[r]) * v1[r];
        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C[0]) + ci) = v0;
        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C[1]) + ci) = v1;
        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C[2]) + ci) = h;
      }
      continue;
    }
    f32x4 out[2];
    int n[2];
    if (B_KC) {
      out[0] = v0; out[1] = v1;
      n[0] = nw + 4 * q; n[1] = nw + 16 + 4 * q;
    } else {
      out[0] = f32x4{v0[0], v1[0], v0[1], v1[1]}; out[1] = f32x4{v0[2], v1[2], v0[3], v1[3]};
      n[0] = nw + 8 * q; n[1] = n[0] + 4;
    }
    float dot = 0.f;
    const float rs = EPI == kEpiDSwiglu ? g.row_scale[m_in ? m : m_end - 1] : 1.f;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      if (!m_in || n[x] >= Ndim) continue;
      const long ci = c_group + m * c_ms + n[x];
      if (EPI == kEpiStore) {
        float* c = reinterpret_cast<float*>(SETS ? st.C : g.C[0]) + ci;
        if (vec) {
          if (g.accumulate) out[x] += *reinterpret_cast<const f32x4*>(c);
          *reinterpret_cast<f32x4*>(c) = out[x];
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (n[x] + r < Ndim) c[r] = g.accumulate ? c[r] + out[x][r] : out[x][r];
        }
      } else {
        const f32x4 a = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.E[0]) + ci);
        const f32x4 b = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.E[1]) + ci);
        f32x4 da, db, hg;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float uu = out[x][r], sg = sigmoidf_(a[r]);
          const float h = a[r] * sg * b[r];
          dot = fmaf(uu, h, dot);
          const float dh = rs * uu;
          hg[r] = rs * h;
          da[r] = dh * b[r] * sg * (1.f + a[r] * (1.f - sg));
          db[r] = dh * a[r] * sg;
        }
        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C[0]) + ci) = da;
        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C[1]) + ci) = db;
        if (store2) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C[2]) + ci) = hg;
      }
    }
    if (EPI == kEpiDSwiglu) {
      // gate-gradient partial of this row over the wavefront's 32 columns, which its four lanes share
      dot += __shfl_xor(dot, 16, kWave);
      dot += __shfl_xor(dot, 32, kWave);
      if (q == 0 && m_in && nw < Ndim) g.rowdot[(long)(nw / plan::kF32RowdotCols) * g.rowdot_stride + m] = dot;
    }
  }
}

typedef Cfg<64, 64, 1, 4> Wide;          // 64 KB of LDS each: two blocks per CU
typedef Cfg<32, 64, 2, 3> Half;          // 72 KB
typedef Cfg<32, 32, 4, 2> Deep;          // 64 KB
static_assert(Wide::BM == plan::kF32Rows && Half::BM == plan::kF32ShortRows && Deep::BM == plan::kF32ShortRows, "the row tiles that the plan counts");

template <int MODE, int EPI, bool A_KC, bool B_KC, bool SETS, typename C>
int launch_tile(const GemmArgs& g, hipStream_t s) {
  constexpr int BNO = EPI == kEpiSwiglu ? C::BN / 2 : C::BN;
  dim3 grid;
  if (MODE == kRaggedM) {
    grid = dim3(cdiv(g.Ndim, BNO), g.max_tiles, 1);
  } else {
    // all tiles of a result along x: the router scores of the most tokens have 131072 row tiles, twice what the other dimensions hold
    int rows[3] = {g.Mdim}, cols[3] = {g.Ndim};
    for (int i = 0; SETS && i < g.n_sets; ++i) { rows[i] = g.set[i].Mdim; cols[i] = g.set[i].Ndim; }
    const long tiles = plan::set_grid_tiles(rows, cols, SETS ? g.n_sets : 1, C::BM, C::BN);
    if (tiles * 256 >= (1L << 32)) return SPES_ESHAPE;   // work-items along a grid dimension
    grid = dim3((unsigned)tiles, 1, g.n_groups * (SETS ? g.n_sets : 1));
  }
  if (grid.x == 0 || grid.y == 0 || grid.z == 0) return SPES_OK;
  hipLaunchKernelGGL((gemm_f32_kernel<MODE, EPI, A_KC, B_KC, SETS, C>), grid, dim3(256), 0, s, g);
  return hipGetLastError() == hipSuccess ? SPES_OK : SPES_EHIP;
}

template <int EPI, bool B_KC>
int launch_ragged(const GemmArgs& g, hipStream_t s) {
  if (g.row_tile == Wide::BM) return launch_tile<kRaggedM, EPI, true, B_KC, false, Wide>(g, s);
  if (g.row_tile != Deep::BM) return SPES_EINVAL;
  // (a fused SwiGLU tile has half as many columns)
  const long blocks = (long)g.est_tiles * cdiv(g.Ndim, EPI == kEpiSwiglu ? Half::BN / 2 : Half::BN);
  if (blocks >= plan::kF32Blocks) return launch_tile<kRaggedM, EPI, true, B_KC, false, Half>(g, s);
  return launch_tile<kRaggedM, EPI, true, B_KC, false, Deep>(g, s);
}

template <bool KC, bool SETS>
int launch_grouped(const GemmArgs& g, hipStream_t s) {
  const long blocks = plan::tiles(g.Mdim, g.Ndim, Wide::BM, Wide::BN) * g.n_groups * (SETS ? g.n_sets : 1);
  if (blocks >= plan::kF32Blocks / 2 && g.Mdim > Deep::BM && g.Ndim > Deep::BN)
    return launch_tile<kGroupedK, kEpiStore, KC, KC, SETS, Wide>(g, s);
  return launch_tile<kGroupedK, kEpiStore, KC, KC, SETS, Deep>(g, s);
}

}  // namespace

// fp32 operands whose 16-byte vectors are aligned (strides that are multiples of four elements) and which 32-bit byte
// offsets cover from the first row of a tile; the caller sees to both (plan::f32_on_matrix_cores)
int launch_gemm_f32(int mode, int epi, bool a_kcontig, bool b_kcontig, const GemmArgs& g, hipStream_t s) {
  if (mode == kRaggedM) {
    if (!a_kcontig) return SPES_EINVAL;
    if (epi == kEpiSwiglu && b_kcontig) return launch_ragged<kEpiSwiglu, true>(g, s);
    if (epi == kEpiStore && b_kcontig) return launch_ragged<kEpiStore, true>(g, s);
    if (epi == kEpiStore && !b_kcontig) return launch_ragged<kEpiStore, false>(g, s);
    if (epi == kEpiDSwiglu && !b_kcontig) return launch_ragged<kEpiDSwiglu, false>(g, s);
    return SPES_EINVAL;
  }
  if (epi != kEpiStore || a_kcontig != b_kcontig) return SPES_EINVAL;
  if (g.n_sets > 0) return a_kcontig ? SPES_EINVAL : launch_grouped<false, true>(g, s);
  return a_kcontig ? launch_grouped<true, false>(g, s) : launch_grouped<false, false>(g, s);
}

}  // namespace spes
