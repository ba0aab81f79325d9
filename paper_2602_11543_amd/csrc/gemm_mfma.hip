// Grouped bf16 GEMM on the gfx950 matrix cores (v_mfma_f32_16x16x32_bf16, fp32 accumulate).
//
// A 256-thread block (four wavefronts, 2 x 2) computes a BM x BN output tile, each
// wavefront a (BM/2) x (BN/2) sub-tile as TM x TN MFMA tiles of 16 x 16 held in AGPRs.
// The 16x16x32 form of the instruction is used because it is the cheaper one in power, and
// power is what bounds these kernels: on the same operand values a register-resident loop of it
// sustains about 2.1 PFLOP/s at 2.1 GHz where the 32x32x16 form sustains 1.85 PFLOP/s at
// 1.83 GHz (it moves half as many accumulator registers per multiply-add).
// Operand tiles go from memory straight into LDS (buffer loads with an LDS destination), K-tiles of 64:
//   * A wavefront issues an instruction every four cycles and an MFMA takes sixteen, and with one wavefront on a SIMD whatever
//     does not fit between two MFMAs is lost.  So fragment reads, loads and the scalars of the next tiles are dealt out over
//     the 128 gaps of a K-tile, one or two to a gap, and the loop is one basic block.
//   * The loads are spread evenly over the whole iteration: the vector-memory path takes a CU's 64 KB of a K-tile at 64 bytes a
//     clock, half an iteration, and a wavefront whose load finds it busy stands still.  Cycles per K-tile of gate + up at 32768
//     tokens 4096 x 1408, 64 experts, 2048 of them MFMAs: a load every second gap 3340, every fourth 2750, every
//     fifth 2560, every eighth 2390 (no load at all 2300).
//   * That leaves a load little time in two LDS slots, so the A operand has a third one where LDS has room (256 x 256 tiles: all
//     160 KB).  With two for both the same loop takes 2740 cycles.
//   * MFMA fragments are double-buffered in registers: the reads of k-step s+1 are issued before the MFMAs of k-step s.
// Against staging through registers (a load, then a write to LDS, for every 16 bytes of a lane) this takes the sixteen LDS
// writes, 64 registers and the waits for them out of a K-tile: 3000 to 3200 cycles before.  The clock under the power cap
// falls as the cycles do (1.82 to 1.73 GHz), so the time gains less: gate + up above 5.48 -> 4.75 ms, its dgrad 5.44 -> 4.65,
// the step 19.3 -> 17.7.
// An operand whose contraction index is the fast memory axis lives in LDS as [row][k], one whose contraction index is the slow
// axis (the weights in the input-gradient GEMMs, both operands of the weight-gradient GEMMs) as [k][row], loaded in
// runs along a k-row; its MFMA fragments (eight consecutive k of one row per lane) come out of LDS through the
// transposing read ds_read_b64_tr_b16, four k at a time.  Both are permuted within a row against bank conflicts (below).
//
// The MFMA operands are swapped (weights tile as the "A" input) so that each lane ends
// up holding runs of four consecutive output columns of one row: epilogues then work
// on 8- and 16-byte vectors along the contiguous dimension.
//
// Tiles are enumerated on a 1-D grid and dealt out so that every XCD (workgroups are
// assigned to the eight XCDs round-robin) gets one contiguous range of tiles: tiles
// that share an expert's weight panel or a row panel meet in the same L2.
#include <type_traits>

#include "gemm.h"
#include "lds_load.h"
#include "plan.h"

namespace spes {
namespace {

constexpr int kXcds = 8;

template <int BM_, int BN_, int NSA_, int NSB_, int MINB_>
struct Cfg {
  static constexpr int BM = BM_, BN = BN_, MINB = MINB_;
  static constexpr int NSA = NSA_, NSB = NSB_;              // LDS slots of each operand, one K-tile each
  static constexpr int BK = 64, KSTEPS = 2;                 // k per K-tile; one MFMA contracts 32
  static constexpr int TM = BM / 32, TN = BN / 32;          // 16 x 16 MFMA tiles per wavefront along m, n
  static constexpr int TS = BM / 64;                        // 32-row slabs of a wavefront's sub-tile (epilogues)
  static constexpr int NA = BM / 32, NB = BN / 32;          // 1 KB loads per wavefront and K-tile
  static constexpr int A_VEC = BM * 8, B_VEC = BN * 8;      // 16-byte units of a slot
  static constexpr int LDS_VEC = NSA * A_VEC + NSB * B_VEC;
};

__device__ __forceinline__ uint32_t pack2(float a, float b) { return pack_bf16x2(a, b); }

constexpr int kGroupRows = 4;      // row tiles per group of the tile order (ragged-row GEMMs) ...
constexpr int kGroupMinCols = 8;   // ... used when the output has at least this many column tiles

// result type of kEpiStore: the router scores and the weight gradients are fp32, the rest has the storage type
constexpr bool f32_out(int mode) { return mode == kGroupedK; }

// 16-byte units of LDS that a tile uses: its operand slots, or the four wavefronts' epilogue slabs (32 padded float rows each) and
// row dots
template <typename C>
constexpr int lds_units() {
  constexpr int slabs = 32 * (C::TN * 16 + 4) + C::BM / 2;
  return C::LDS_VEC > slabs ? C::LDS_VEC : slabs;
}

// an element at an address that is the same for the whole wavefront, of a table that an earlier launch wrote, requested where this stands
__device__ __forceinline__ int scalar_load(const int* p) { return *(__attribute__((address_space(4))) const volatile int*)(unsigned long)p; }

// Tile `block` of `total`, dealt out so that every XCD (workgroups go round the eight) gets one contiguous range; none: total or more
__device__ __forceinline__ unsigned dealt(unsigned block, unsigned total) {
  const unsigned per_xcd = (total + kXcds - 1) / kXcds, slot = block / kXcds;
  return slot < per_xcd ? (block % kXcds) * per_xcd + slot : total;
}

// One tile.  block: ragged rows: the tile's number among the column tiles of mt_count row tiles, which stand in the table from mt_first on;
// otherwise the position in the launch.  half: the lower half of a full entry of the table
// SETS: several contractions over the same groups in one launch (the three weight gradients), each with its own operands
// and result; either operand of a set may take its k-rows through the index table k_rows (the dy rows, or the input
// rows, of an expert's routed pairs)
// GATHER: which operand of a set (1 A, 2 B) takes its k-rows through the index table
template <int MODE, int EPI, bool A_KC, bool B_KC, bool SETS, typename C, int GATHER = 0>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, uint4* const smem, const unsigned block, const int mt_first, const int mt_count, const int half = 0) {
  constexpr int BM = C::BM, BN = C::BN, BK = C::BK, TM = C::TM, TN = C::TN, NSA = C::NSA, NSB = C::NSB;
  constexpr int A_VEC = C::A_VEC, B_VEC = C::B_VEC;
  const int tid = threadIdx.x, lane = tid & 63, wave = (int)uniform(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;          // an MFMA operand: lane holds row l16, k = lq*8 .. lq*8+7 of a 32-wide k-step
  const int wm = wave >> 1, wn = wave & 1;
  constexpr int BNO = (EPI == kEpiSwiglu) ? BN / 2 : BN;   // output columns per tile
  constexpr bool F32_OUT = f32_out(MODE);

  // ---- which tile ----
  // What is ahead of a tile's first MFMA is a chain of round trips (number of tiles, tile table, expert's end and index table, operands) with
  // integer divisions between them, and nothing else runs on the CU.  The scalars come in pairs, the divisions are 32-bit, the
  // weights' first K-tile, which needs no index, is requested before the indices are waited for, and the indices come by
  // scalar loads, which do not wait in line with it.  From a tile's start to its operand loads 1.3 us, and 2.8 in a launch's first round;
  // now 0.5 to 1.0, and 0.8.  With the surplus rows' fetches left out as well: steps of 1531 tokens 512 x 352 153 -> 145 us, 4096
  // tokens 768 x 2048 479 -> 469, 3777 tokens 1536 x 1280 328 -> 318, 16384 tokens 2048 x 1024 3854 -> 3818.
  const int n_base = MODE == kRaggedM ? g.n_base : 0;
  int Mdim = g.Mdim, Ndim = g.Ndim;
  unsigned gx = (unsigned)(Ndim - n_base + BNO - 1) / BNO;
  // (32-bit: a launch has fewer blocks, and a 64-bit division takes a wavefront some 700 cycles)
  unsigned logical = block;
  if (MODE == kGroupedK) {
    const unsigned total = (unsigned)g.n_groups * ((unsigned)(Mdim + BM - 1) / BM) * gx * (SETS ? (unsigned)g.n_sets : 1u);
    // ragged contraction lengths: tiles are taken in block order (round-robin over the XCDs) and the groups are
    // visited longest first, so the long tiles start early and the short ones fill in behind them
    if (g.offset == nullptr) logical = dealt(block, total);
    if (logical >= total) return;
  }
  int set = 0;
  if (SETS) {
    // the sets of a group stand side by side, all of the longest group's tiles first; a set whose result is the
    // transposed shape has the same number of (square) tiles
    const unsigned per_set = (unsigned)cdiv(Mdim, BM) * gx, at = logical;
    const unsigned pos = at / per_set, grp_pos = pos / 3u;       // three sets (see launch); 32-bit: a grid has fewer blocks
    set = (int)(pos - grp_pos * 3u);
    logical = grp_pos * per_set + (at - pos * per_set);
    Mdim = g.set[set].Mdim; Ndim = g.set[set].Ndim;
    gx = (unsigned)(Ndim + BNO - 1) / BNO;
  }
  const void* const opA0 = SETS ? g.set[set].A : g.A[0];
  const void* const opB0 = SETS ? g.set[set].B : g.B[0];
  void* const opC0 = SETS ? g.set[set].C : g.C[0];
  const long a_ks = SETS ? g.set[set].a_ks : g.a_ks, b_ks = SETS ? g.set[set].b_ks : g.b_ks;
  const long c_ms = SETS ? g.set[set].c_ms : g.c_ms;
  static_assert(SETS == (GATHER != 0), "one operand of every set");
  constexpr bool a_gather = GATHER == 1, b_gather = GATHER == 2;
  unsigned nt, mt_all;
  if (MODE == kRaggedM && gx >= kGroupMinCols) {
    // Row tiles are taken kGroupRows at a time and the column tiles run inside such a group, so that the 32 tiles an
    // XCD works on at once are about kGroupRows row panels times 32/kGroupRows column panels: with the plain
    // row-major order a wide output (many column tiles) has every CU of the XCD stream its own weight panel, and the
    // next row tile of the expert streams them all again.
    const unsigned per_group = kGroupRows * gx;
    const unsigned grp_i = logical / per_group, within = logical - grp_i * per_group;
    const unsigned left = (unsigned)mt_count - grp_i * kGroupRows;
    if (left >= kGroupRows) {
      nt = within / kGroupRows;
      mt_all = grp_i * kGroupRows + within % kGroupRows;
    } else {
      nt = within / left;
      mt_all = grp_i * kGroupRows + (within - nt * left);
    }
  } else {
    mt_all = logical / gx;
    nt = logical - mt_all * gx;
  }
  if (MODE == kRaggedM) mt_all += (unsigned)mt_first;

  long m0, m_end, k_begin, k_end, b_group = 0, c_group = 0;
  // kRaggedM with gathered rows of A (every row read from x or dy): the index table's entries of this wavefront's rows, eight per load of
  // a K-tile, four loads at a time in scalar registers, where they do not wait in line with the loads into LDS.  (Entries beyond
  // the tile's last row are there to be read, at worst in the regions of the context behind the table, and not used.)
  constexpr bool ROWS = MODE == kRaggedM && EPI != kEpiStore;
  constexpr int ROWB = C::NA < 4 ? C::NA : 4;
  typedef __attribute__((ext_vector_type(8))) int i32x8;
  typedef __attribute__((address_space(4))) const i32x8 const_i32x8 __attribute__((aligned(4)));
  i32x8 row_idx[ROWB];
  auto request_rows = [&](int first) {
    if (ROWS) {
#pragma unroll
      for (int i = 0; i < ROWB; ++i) row_idx[i] = *(volatile const_i32x8*)(unsigned long)(g.a_rows + (int)uniform((unsigned)m0 + (unsigned)wave * 8 + 32u * (unsigned)(first + i)));
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  bool ds_store2 = true;
  if (MODE == kRaggedM) {
    // (each pair of scalar loads together: one round trip)
    int e = scalar_load(g.tile_expert + mt_all), row0 = scalar_load(g.tile_row0 + mt_all);
    asm volatile("" : "+s"(e), "+s"(row0));
    ds_store2 = ((g.c2_skip >> e) & 1ull) == 0;
    m0 = row0 + half * plan::kHalfRows;
    const int end = scalar_load(g.offset + e + 1);
    request_rows(0);
    m_end = min((long)end, m0 + BM);
    k_begin = 0; k_end = g.Kdim;
    b_group = (long)e * g.b_gs;
  } else {
    const unsigned my = (unsigned)cdiv(Mdim, BM);
    int grp = (int)(mt_all / my);
    m0 = (long)(mt_all - (unsigned)grp * my) * BM;
    m_end = min((long)Mdim, m0 + BM);
    if (g.offset != nullptr) {
      // grp counts positions in descending order of length; find the group that holds this position
      // (lane e owns expert e; ties go to the lower group, so the order is a permutation).  One round trip, and lane reads instead of
      // shuffles: with the index entries ahead of their loads, 1.5 to 2.7 -> 1.1 to 2.0 us from a tile's start to its first load; steps of
      // 4096 tokens 2048 x 2048, 8 of 32 experts, accumulating 1208 -> 1190 us, 3777 tokens 1536 x 1280 314 -> 310, 4096 tokens 768 x 2048 469 -> 464.
      const int first = g.offset[lane < g.n_experts ? lane : 0], mine = g.offset[lane < g.n_experts ? lane + 1 : 0] - first;
      int rank = 0;
      for (unsigned long long rest = g.groups; rest != 0; rest &= rest - 1) {
        const int j = __builtin_ctzll(rest), other = __builtin_amdgcn_readlane(mine, j);
        rank += (other > mine || (other == mine && j < lane)) ? 1 : 0;
      }
      const unsigned long long hit = __ballot((g.groups >> lane & 1) != 0 && rank == grp);
      const int e = __builtin_ctzll(hit);
      grp = __builtin_popcountll(g.groups & ((1ull << e) - 1));
      k_begin = __builtin_amdgcn_readlane(first, e);
      k_end = k_begin + __builtin_amdgcn_readlane(mine, e);
    } else {
      k_begin = (long)grp * g.kchunk; k_end = min((long)g.Kdim, k_begin + g.kchunk);
    }
    c_group = (long)grp * g.c_gs;
  }
  const long n0 = n_base + (long)nt * BNO;

  // ---- operands are read through buffer resources whose base moves with the K-tile; a lane's byte offsets are fixed for the
  // whole tile (but for gathered k-rows).  The resource ends where the operand does, or, for a K-strided one, where the contraction
  // range does, so k beyond the range, rows beyond the tensor and whole K-tiles beyond the last one come back as zeros
  // without a fetch.  Rows inside the tensor but outside the tile bring data that is never stored.
  const int klen = (int)uniform((unsigned)(k_end - k_begin));
  const int npass = (EPI == kEpiSwiglu) ? 1 : g.npairs;
  const int nk = klen > 0 ? (klen + BK - 1) / BK : 1;       // an empty range: one K-tile of zeros
  const int nsteps = nk * npass;
  const unsigned a_step = uniform(A_KC ? 2u : a_gather ? 0u : (unsigned)(a_ks * 2));       // bytes per k
  const unsigned b_step = uniform(B_KC ? 2u : b_gather ? 0u : (unsigned)(b_ks * 2));
  auto base_of = [&](const void* p, long elems) -> unsigned long {
    const unsigned long v = reinterpret_cast<unsigned long>(p) + (unsigned long)(elems * 2);
    return (unsigned long)uniform((unsigned)(v >> 32)) << 32 | uniform((unsigned)v);
  };
  const long a_first = A_KC ? k_begin : a_gather ? 0 : k_begin * a_ks, b_first = b_group + (B_KC ? k_begin : b_gather ? 0 : k_begin * b_ks);
  const unsigned long a_base0 = base_of(opA0, a_first), a_base1 = base_of(!SETS && g.A[1] ? g.A[1] : opA0, a_first);
  const unsigned long b_base0 = base_of(opB0, b_first), b_base1 = base_of(!SETS && g.B[1] ? g.B[1] : opB0, b_first);
  const unsigned a_bytes = uniform(A_KC || a_gather ? (unsigned)(((SETS ? g.set[set].a_elems : g.a_elems) - a_first) * 2) : (unsigned)klen * a_step);
  const unsigned b_bytes = uniform(B_KC || b_gather ? (unsigned)(((SETS ? g.set[set].b_elems : g.b_elems) - b_first) * 2) : (unsigned)klen * b_step);

  // LDS layout of a K-contiguous operand: [row][k], 128 bytes a row, the eight 16-byte chunks of a row permuted by the row
  // number (chunk c of row r at position c ^ (r >> 1 & 7)), so that the sixteen rows a group of sixteen lanes reads at a common
  // chunk cover all banks.  The permutation is made on the way in: a load's lanes are eight rows by eight positions, and each
  // lane asks for the chunk that belongs at its position.
  const int kc_chunk = (lane & 7) ^ ((wave * 4 + (lane >> 4)) & 7);
  // A K-strided operand keeps its memory order, [k][row] without padding; the chunks of a k-row are permuted by twice the
  // low two bits of k, so that the four k-rows of 32 bytes that one group of lanes reads with the transposing read cover all banks.
  // The four wavefronts' loads i stand side by side; with k-rows from the index table a wavefront's loads stand one behind the
  // other, so that its sixteen k-rows are sixteen entries of the table in a row.  Either way k-row r of a slot is the K-tile's k = r: the
  // sums have one order on every tile, and an expert's gradients do not change with the tile that the number of trainable
  // experts decides.
  constexpr int ACH = BM / 8, BCH = BN / 8;       // 16-byte chunks per k-row
  constexpr unsigned LOAD_STEP = SETS ? 1024u : 4096u;       // bytes in LDS from one load of a wavefront to its next
  auto ks_k = [&](int i, int ch, int n) { return SETS ? wave * 16 + i * (16 / n) + lane / ch : wave * (64 / ch) + lane / ch + i * (64 / n); };
  auto ks_col = [&](int i, int ch, int n, long first) { return (unsigned)((first + (((lane % ch) ^ (2 * (ks_k(i, ch, n) & 3))) * 8)) * 2); };
  auto ks_off = [](unsigned long o) { return o < kOutOfRange ? (unsigned)o : kOutOfRange; };   // k-rows beyond a short, wide operand
  unsigned aoff[C::NA], boff[C::NB];
  // of A: kRaggedM, once the first loads of B are on their way, ROWB loads at a time; surplus rows: zeros, without a fetch
  auto ragged_rows = [&](int first) {
    if (ROWS) {
#pragma unroll
      for (int i = 0; i < ROWB; ++i) asm volatile("" : "+s"(row_idx[i]));
    }
#pragma unroll
    for (int i = 0; i < ROWB; ++i) {
      const int m = (int)m0 + wave * 8 + (lane >> 3) + 32 * (first + i);
      int row = m;
      if (ROWS) {
        row = row_idx[i][0];
#pragma unroll
        for (int h = 1; h < 8; ++h) row = lane >> 3 == h ? row_idx[i][h] : row;
      }
      aoff[first + i] = m < (int)m_end ? ((unsigned)row * (unsigned)g.a_ms + (unsigned)kc_chunk * 8u) * 2u : kOutOfRange;
    }
  };
  if (!A_KC) {
#pragma unroll
    for (int i = 0; i < C::NA; ++i) aoff[i] = ks_off(ks_k(i, ACH, C::NA) * a_ks * 2 + ks_col(i, ACH, C::NA, m0));
  } else if (MODE != kRaggedM) {
#pragma unroll
    for (int i = 0; i < C::NA; ++i) aoff[i] = (unsigned)(((m0 + wave * 8 + (lane >> 3) + 32 * i) * g.a_ms + kc_chunk * 8) * 2);
  }
  // fused SwiGLU: load i brings rows of the gate matrix (B[0]) or of the up matrix (B[1]); tile row nl -> wave column, then
  // (BN/4) gate columns followed by the matching (BN/4) up columns
  constexpr int SW_W = BN / 2, SW_H = BN / 4;
  static_assert(EPI != kEpiSwiglu || (SW_H % 32 == 0), "a load must not straddle the gate / up boundary");
#pragma unroll
  for (int i = 0; i < C::NB; ++i) {
    if (B_KC) {
      const int nl = wave * 8 + (lane >> 3) + 32 * i;
      const long col = (EPI == kEpiSwiglu) ? n0 + (nl / SW_W) * SW_H + (nl % SW_H) : n0 + nl;
      boff[i] = (unsigned)((col * g.b_ns + kc_chunk * 8) * 2);
    } else {
      boff[i] = ks_off(ks_k(i, BCH, C::NB) * b_ks * 2 + ks_col(i, BCH, C::NB, n0));
    }
  }

  // acc[j][i][r] = C(m = i*16 + l16, n = j*16 + lq*4 + r) of the wavefront's sub-tile
  f32x4 acc[TN][TM];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[j][i][r] = 0.f;
  // (zeros that the compiler takes for different values: from one common zero it starts the loop with accumulators that it then
  // moves to their places in every iteration)
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (C::MINB == 1) asm("" : "+a"(acc[j][i]));
      else asm("" : "+v"(acc[j][i]));
    }

  // ---- the K-tiles being loaded (numbers la, lb; the tiles of all passes in a row) ----
  constexpr int NA = C::NA, NB = C::NB, NP = NA + NB;
  constexpr bool TWO_PASS = MODE == kRaggedM && EPI == kEpiStore && !B_KC;      // the one launch with two operand pairs
  const unsigned lds0 = (unsigned)(unsigned long)(__attribute__((address_space(3))) uint4*)smem + (unsigned)wave * (SETS ? NA * 1024u : 1024u);
  struct Src { unsigned lo, hi, bytes, left, dst; };     // resource base and size; k left from the tile's first one on; LDS address
  Src as = {0, 0, 0, 0, 0}, bs = as;
  // Every block takes the K-tiles in their order, so that a result's bits follow from its operands and not from the place of its
  // tile or the number of its expert (copies of an expert, and its gate gradients, stay equal).  Blocks that start together then walk
  // down the same 128 bytes of every row of K-contiguous weights, which with rows a power of two apart are the same few memory channels.
  // A start of its own for each XCD or each expert avoids that (200 tokens, 32 experts of 2048 x 2048, top-4: forward 161 us against
  // 232; 4096 tokens 1 %, longer launches nothing), but adds up equal rows in different orders.
  unsigned b1_lo = 0, b1_hi = 0;                         // fused SwiGLU: the base in the second matrix
  // in steps, so that the main loop can deal them out: 0 the k, 1 the base, 2 the size, 3 where to
  auto next_src = [&](Src& x, int step, int lt, unsigned per_k, unsigned long base0, unsigned long base1, unsigned bytes, unsigned dst) {
    const bool second = TWO_PASS && lt >= nk;
    if (step == 0) {
      x.left = (unsigned)(klen - (lt - (second ? nk : 0)) * BK);
      pin(x.left);
    } else if (step == 1) {
      const unsigned long at = (second ? base1 : base0) + ((unsigned)klen - x.left) * per_k;
      x.lo = (unsigned)at; x.hi = (unsigned)(at >> 32);
      pin(x.lo); pin(x.hi);
    } else if (step == 2) {
      x.bytes = lt < nsteps ? bytes - ((unsigned)klen - x.left) * per_k : 0u;
      pin(x.bytes);
    } else {
      x.dst = dst;
      pin(x.dst);
    }
  };
  auto next_a = [&](int step, int la, int slot) {
    next_src(as, step, la, a_step, a_base0, a_base1, a_bytes, lds0 + (unsigned)slot * (A_VEC * 16u));
  };
  auto next_b = [&](int step, int lb, int slot) {
    next_src(bs, step, lb, b_step, b_base0, b_base1, b_bytes, lds0 + NSA * A_VEC * 16u + (unsigned)slot * (B_VEC * 16u));
    if (EPI == kEpiSwiglu && step == 1) {
      const unsigned long at = b_base1 + ((unsigned)klen - bs.left) * b_step;
      b1_lo = (unsigned)at; b1_hi = (unsigned)(at >> 32);
      pin(b1_lo); pin(b1_hi);
    }
  };
  // The index table's entries of a wavefront's sixteen k-rows, in scalar registers: requested an iteration before they are needed,
  // while no LDS read is outstanding (both count on one counter, out of order), and turned into offsets one load at a time.
  // Entries beyond the range are there to be read (up to 63, see GemmArgs) and not used: their loads are masked.  (As loads
  // of each lane's own indices, waited for in order behind the loads into LDS, they emptied the memory queue in every
  // K-tile, and their 64-bit addresses, clamps and selects were two thirds of 224 vector instructions a K-tile, now 57:
  // 1024 rows an expert, 3584 x 4864, 4100 -> 3000 cycles per K-tile, the launch 1228 -> 1050 us.)
  typedef __attribute__((ext_vector_type(16))) int i32x16;
  typedef __attribute__((address_space(4))) const i32x16 const_i32x16 __attribute__((aligned(4)));
  i32x16 kidx, kidx_next;
  auto load_kidx = [&](int lt) {
    if (SETS) {
      const int at = (int)uniform((unsigned)k_begin) + (lt < nsteps ? lt : nsteps - 1) * BK + wave * 16;
      kidx_next = *(volatile const_i32x16*)(unsigned long)(g.k_rows + at);
    }
  };
  auto have_kidx = [&]() {
    if (SETS) { asm volatile("" : "+s"(kidx_next)); kidx = kidx_next; }
  };
  auto take_kidx = [&](int j) {
    if (SETS) {
      constexpr int CHK = a_gather ? ACH : BCH, RPL = 64 / CHK;       // k-rows per load
      int row = kidx[j * RPL];
#pragma unroll
      for (int h = 1; h < RPL; ++h) row = lane / CHK == h ? kidx[j * RPL + h] : row;
      if (a_gather) aoff[j] = (unsigned)row * (unsigned)(a_ks * 2) + ks_col(j, ACH, NA, m0);
      if (b_gather) boff[j] = (unsigned)row * (unsigned)(b_ks * 2) + ks_col(j, BCH, NB, n0);
    }
  };
  // load p of a K-tile, B first, in two steps; `masked`: the tile may reach beyond the contraction range of K-contiguous operands
  unsigned lds_dest = 0;
  auto aim = [&](int p) { lds_dest = set_lds_dest(p < NB ? bs.dst + (unsigned)p * LOAD_STEP : as.dst + (unsigned)(p - NB) * LOAD_STEP); };
  auto load = [&](int p, bool masked) {
    if (p < NB) {
      const int kb = B_KC ? kc_chunk * 8 : ks_k(p, BCH, NB);
      const unsigned off = (B_KC || b_gather) && masked && kb >= (int)bs.left ? kOutOfRange : boff[p];
      // (the load -> matrix assignment of the fused SwiGLU is the same for every thread)
      const bool up = EPI == kEpiSwiglu && ((32 * p) % SW_W) / SW_H != 0;
      load_to_lds(rsrc_t{up ? b1_lo : bs.lo, up ? b1_hi : bs.hi, bs.bytes, 0x00020000u}, off, lds_dest);
    } else {
      const int ka = A_KC ? kc_chunk * 8 : ks_k(p - NB, ACH, NA);
      const unsigned off = (A_KC || a_gather) && masked && ka >= (int)as.left ? kOutOfRange : aoff[p - NB];
      load_to_lds(rsrc_t{as.lo, as.hi, as.bytes, 0x00020000u}, off, lds_dest);
    }
  };

  bf16x8 fa[2][TM], fb[2][TN];
  // fragment addresses within a slot: K-contiguous, chunk ks*4 + lq of row l16 (+ 16 i); K-strided, k-row ks*32 + lq*8 + l16/4
  // (+ 4), columns (lane&3)*4 of the 16-row group u = first group + i, which stands at position u ^ (l16/4) of its four
  const int kc_pos = lq ^ (l16 >> 1);
  const uint4* const a_kc = smem + (wm * (BM / 2) + l16) * 8;
  const uint4* const b_kc = smem + NSA * A_VEC + (wn * (BN / 2) + l16) * 8;
  const bf16_t* const a_tr = reinterpret_cast<const bf16_t*>(smem) + (lq * 8 + (l16 >> 2)) * BM + (lane & 3) * 4 + wm * (BM / 2);
  const bf16_t* const b_tr = reinterpret_cast<const bf16_t*>(smem + NSA * A_VEC) + (lq * 8 + (l16 >> 2)) * BN + (lane & 3) * 4 + wn * (BN / 2);
  static_assert((A_KC || BM >= 128) && (B_KC || BN >= 128), "a wavefront's groups of a K-strided operand start at a multiple of four");
  auto tr_pos = [&](int i) { return (i & ~3) * 16 + ((i & 3) ^ (l16 >> 2)) * 16; };
  auto read_frag_a = [&](int slot, int ks, int set_, int i) {
    if (A_KC) {
      fa[set_][i] = __builtin_bit_cast(bf16x8, a_kc[slot * A_VEC + i * 128 + (kc_pos ^ (ks * 4))]);
    } else {
      const bf16_t* p = a_tr + slot * (A_VEC * 8) + ks * 32 * BM + tr_pos(i);
      const uint2 lo = lds_read_tr(p), hi = lds_read_tr(p + 4 * BM);
      fa[set_][i] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
    }
  };
  auto read_frag_b = [&](int slot, int ks, int set_, int j) {
    if (B_KC) {
      fb[set_][j] = __builtin_bit_cast(bf16x8, b_kc[slot * B_VEC + j * 128 + (kc_pos ^ (ks * 4))]);
    } else {
      const bf16_t* p = b_tr + slot * (B_VEC * 8) + ks * 32 * BN + tr_pos(j);
      const uint2 lo = lds_read_tr(p), hi = lds_read_tr(p + 4 * BN);
      fb[set_][j] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
    }
  };
  // fragment w of a k-step in the order the MFMAs first need them: B0, A0 .. A(TM-1), B1 .. B(TN-1)
  auto read_frag = [&](int sa, int sb, int ks, int set_, int w) {
    if (w == 0) read_frag_b(sb, ks, set_, 0);
    else if (w <= TM) read_frag_a(sa, ks, set_, w - 1);
    else read_frag_b(sb, ks, set_, w - TM);
  };

  // ---- schedule: positions are gaps between the 2 MF MFMAs of a K-tile ----
  // dSwiGLU epilogue: row groups of a wavefront, and how many of them have their a, b and correction requested ahead
  constexpr int ECOLS = TN * 16, DS_CPR = ECOLS / 8, DS_RPI = 64 / DS_CPR, DS_UNITS = BM / 2 / DS_RPI;
  constexpr int DS_AHEAD = DS_UNITS < 8 ? DS_UNITS : C::MINB == 1 ? 8 : 4;
  enum { kPlainLoads, kMaskedLoads, kNextToLast, kLast };          // iterations
  constexpr int MF = TM * TN;                       // MFMAs per k-step
  constexpr int NF = TM + TN;                       // fragments per k-step
  constexpr bool WIDE = MF >= 32;          // room for a second meeting point
  constexpr int F0 = MF >= 64 ? 2 : 1;              // gaps per fragment
  constexpr int QF = NF * F0 + 8 < MF ? NF * F0 + 8 : MF;          // K-tile t is in registers: its slots may be overwritten
  constexpr int QL = WIDE ? 2 * MF - NF * F0 - (MF >= 64 ? 12 : 6) : QF;    // K-tile t+1 is in LDS: its first fragments may be read
  // gaps per load: spread over the whole iteration (A's loads run on into the next one, up to its QF), B's done at its end
  constexpr int DG_ALL = 2 * MF / NP, DG_B = (2 * MF - QF) / NB, DG = DG_ALL < DG_B ? DG_ALL : DG_B;
  constexpr int R0 = QL < MF ? MF : QL;             // the first fragments of K-tile t+1 follow, once their registers are free
  constexpr int F1 = (2 * MF - R0) / NF < 4 ? (2 * MF - R0) / NF : 4;
  constexpr int KG = MF >= 32 ? 2 : 1;              // gaps per offset of gathered k-rows of A
  static_assert(!SETS || !WIDE || QF + KG * NA < MF, "before the next indices replace these");
  constexpr int SS = MF >= 32 ? 2 : 1;              // gaps per step of the scalars of the tiles to be loaded
  static_assert(DG >= 1 && F1 >= 1 && QF + NB * DG <= 2 * MF && R0 + NF * F1 <= 2 * MF && QF >= 4 * SS && NB * DG >= 4 * SS, "more fragments or loads than MFMA gaps");
  constexpr int LATE = QF + NP * DG > 2 * MF ? (QF + NP * DG - 2 * MF + DG - 1) / DG : 0;      // loads of an iteration that the next one issues
  constexpr int LOADED = QL > QF ? ((QL - QF) / DG < NP ? (QL - QF) / DG : NP) : 0;     // loads an iteration has issued before QL
  // loads that may be outstanding at QL, counted back from the last one of K-tile t+1 (B: NSB tiles ahead, A: NSA, behind it)
  constexpr int AFTER_A = (NSA - 2) * NP, AFTER_B = NA + (NSB - 2) * NP;
  constexpr int AHEAD = (AFTER_A < AFTER_B ? AFTER_A : AFTER_B);
  static_assert(AHEAD + NP < 64, "the counter of outstanding loads");
  constexpr bool EARLY = EPI == kEpiDSwiglu;        // an epilogue that reads: its first loads before the main loop ends ...
  constexpr int EG = 4 * MF / (DS_AHEAD * 3);       // ... and the gaps from one of them to the next

  // prologue: the first NSA and NSB K-tiles, in the order in which the iterations -NS .. -1 would have loaded them
  constexpr int FAR = NSA > NSB ? NSA : NSB, NEAR = NSA > NSB ? NSB : NSA, NSG = a_gather ? NSA : NSB;
  if (MODE == kRaggedM) {
#pragma unroll
    for (int st = 0; st < 4; ++st) next_b(st, 0, 0);
#pragma unroll
    for (int p = 0; p < NB; ++p) { aim(p); one_instruction(); load(p, true); }
#pragma unroll
    for (int st = 0; st < 4; ++st) next_a(st, 0, 0);
#pragma unroll
    for (int first = 0; first < NA; first += ROWB) {
      ragged_rows(first);
      if (first + ROWB < NA) request_rows(first + ROWB);
#pragma unroll
      for (int p = NB + first; p < NB + first + ROWB; ++p) { aim(p); one_instruction(); load(p, true); }
    }
  }
  if (FAR == NSG) load_kidx(0);
#pragma unroll
  for (int u = -FAR; u < 0; ++u) {
    if (SETS && u + NSG >= 0) {
      have_kidx();
#pragma unroll
      for (int j = 0; j < (a_gather ? NA : NB); ++j) take_kidx(j);
    }
    load_kidx(u + 1 + NSG);                            // (by the time they are needed; the last ones are the first iteration's)
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      if (u + NSB >= (MODE == kRaggedM ? 1 : 0)) next_b(st, u + NSB, u + NSB);
      if (u + NSA >= (MODE == kRaggedM ? 1 : 0)) next_a(st, u + NSA, u + NSA);
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if ((p < NB ? u + NSB : u + NSA) < (MODE == kRaggedM ? 1 : 0) || (u == -1 && p >= NP - LATE)) continue;
      aim(p); one_instruction(); load(p, true);
    }
  }
  wait_and_meet<AHEAD + NP - LATE>();
  have_kidx();
#pragma unroll
  for (int w = 0; w < NF; ++w) read_frag(0, 0, 0, 0, w);

  // One iteration: the MFMAs of K-tile t, whose first fragments are in registers.  Before QF: the fragments of its second k-step,
  // and the scalars of the tiles to be loaded.  At QF the wavefronts meet: K-tile t is in registers everywhere, and its slots are
  // loaded anew, one load every DG gaps.  At QL they meet again: K-tile t+1 is in LDS everywhere; its first fragments follow.
  // A wavefront issues an instruction every four cycles and an MFMA takes sixteen, so a gap has room for three others: they are
  // dealt out one or two to a gap.  No branches in here: past the last K-tile the loads bring zeros, and the fragments are
  // never used.
  // `behind`: the last two iterations of a launch with EARLY epilogue loads, which load no K-tile but call behind(gap).
  auto iteration = [&](int t, int sa, int sb, int sa1, int sb1, auto kind_c, auto behind) __attribute__((always_inline)) {
    constexpr int KIND = decltype(kind_c)::value;
    constexpr bool MASKED = KIND == kMaskedLoads, LOADS = KIND <= kMaskedLoads;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 2 * MF; ++q) {
      const int ks = q / MF, j = (q % MF) / TM, i = q % TM;
      if (q == QF && LOADS) {
        wait_and_meet<(WIDE ? 63 : AHEAD)>();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (WIDE && q == QL && LOADS) {
        wait_and_meet<AHEAD + LOADED>();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (q == QL && KIND == kNextToLast) {
        wait_and_meet<(QL + EG - 1) / EG>();
        __builtin_amdgcn_sched_barrier(0);
      }
      acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][j], fa[ks][i], acc[j][i], 0, 0, 0);
      if (!LOADS) behind(q);
      if (q < MF && q % F0 == 0 && q / F0 < NF) read_frag(sa, sb, 1, 1, q / F0);
      if (KIND != kLast && q >= R0 && (q - R0) % F1 == 0 && (q - R0) / F1 < NF) read_frag(sa1, sb1, 0, 0, (q - R0) / F1);
      if (LOADS && q >= QF - 4 * SS && q < QF && (QF - 1 - q) % SS == 0) next_b((q - (QF - 4 * SS)) / SS, t + NSB, sb);
      if (LOADS && q >= QF && q < QF + 4 * SS && (q - QF) % SS == 0) next_a((q - QF) / SS, t + NSA, sa);
      // offsets of the gathered operand: B's before its loads begin at QF, A's between the late loads of the tile before and its
      // own; then the next tile's indices, to be here before the next LDS read
      if (b_gather && q >= QF - NB && q < QF) take_kidx(q - (QF - NB));
      if (a_gather && q >= QF && q < QF + KG * NA && (q - QF) % KG == 0) take_kidx((q - QF) / KG);
      if (SETS && q == (WIDE ? QF + 1 : NF * F0 + 1)) load_kidx(t + 1 + NSG);
      if (SETS && q == (WIDE ? MF - 1 : QF + NA)) have_kidx();
      {
        const int at = q >= QF ? q - QF : q - QF + 2 * MF, p = at / DG;
        if (LOADS && p < NP && (q >= QF || p >= NP - LATE)) {
          // (a gap ahead of the load, but in the same iteration)
          const bool alone = DG == 1 || (q == 0 && at % DG == DG - 1);
          if (alone || (at % DG == DG - 2 && q < 2 * MF - 1)) aim(p);
          if (alone) one_instruction();
          if (at % DG == DG - 1) load(p, MASKED);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // The iterations that load the last K-tile of a pass of K-contiguous operands zero what lies beyond the range; they run in a copy of
  // their own, so that the others carry no selects.
  int t = 0, sa = 0, sb = 0;
  auto step = [&](auto kind_c, auto behind) __attribute__((always_inline)) {
    const int sa1 = sa + 1 == NSA ? 0 : sa + 1, sb1 = sb + 1 == NSB ? 0 : sb + 1;
    iteration(t, sa, sb, sa1, sb1, kind_c, behind);
    sa = sa1; sb = sb1;
    ++t;
  };
  auto nothing = [](int) {};
  // the last two iterations of an EARLY launch run behind these (of a single K-tile, the second one multiplies the zeros that follow it):
  // by then every K-tile has been requested, A's NSA = 3 ahead and B's two or three
  const int n_main = EARLY ? (nsteps > 2 ? nsteps - 2 : 0) : nsteps;
  if constexpr (A_KC || B_KC || SETS) {
    int last = klen % BK != 0 ? nk - 1 : nsteps + FAR;        // the next K-tile that needs it
    while (last + 1 < NEAR) last += nk;
    while (true) {
      const int stop = last - FAR < n_main ? last - FAR : n_main;
      while (t < stop) step(std::integral_constant<int, kPlainLoads>{}, nothing);
      if (t >= n_main) break;
      step(std::integral_constant<int, kMaskedLoads>{}, nothing);
      if (t > last - NEAR + 1) last += nk;
    }
  } else {
    do step(std::integral_constant<int, kPlainLoads>{}, nothing); while (t < nsteps);
  }
  if (!EARLY) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // no load may still write the LDS that the epilogue uses

  // ---- epilogue ----
  // The MFMA leaves each lane with 4-column runs of one row per register group, which would scatter 32-byte
  // pieces over 32 rows per store.  Each wavefront therefore turns its sub-tile through a private LDS region,
  // 32 rows at a time, and comes back with lanes laid along the columns: every global access below is a run of
  // 256 to 512 contiguous bytes per row.
  constexpr int EPITCH = ECOLS + 4;                  // floats per LDS row
  constexpr int TS = C::TS;                          // 32-row slabs: slab i holds the MFMA row tiles 2i and 2i+1
  float* ep = reinterpret_cast<float*>(smem) + wave * (32 * EPITCH);
  // output addresses are a per-tile base (uniform) plus a 32-bit element offset: row within the tile times the row
  // stride plus the column; rows are compared with the tile's valid row count in 32 bits as well
  const int e_rows = (int)(m_end - m0);
  const long e_tile = c_group + m0 * c_ms;
  const int e_r0 = wm * (BM / 2);
  // dSwiGLU epilogue: lanes lie along the columns (DS_CPR lanes per row, eight columns each, so that the bf16 results leave in
  // 16-byte stores), DS_RPI rows at a time.  Its loads and stores go through buffer resources that begin at the tile and end with its
  // last row: a lane out of the tile asks for an offset beyond them, so all are unconditional, and the compiler, which knows how many are
  // outstanding, does not wait for stores where it needs a load.  A tile is 5200 vector instructions per wavefront (25 000 cycles), 384 KB in and 256 or
  // 384 KB out (3.5 and 1.9 us where one CU does it alone, 12 and 7 where all do at once).  The first loads go out before the main
  // loop ends, and in the middle of the arithmetic one or two at a time; nothing is formed of gate * h for an expert that does not train.  Before (batches of 12 loads
  // and 12 stores, each load waited for behind the stores before it) the half-width tiles took 22 800 cycles, now 18 600: steps of
  // 1531 tokens 512 x 352 163 -> 161 us, 4096 tokens 768 x 2048 489 -> 484, 3777 tokens 1536 x 1280 331 -> 327, 16384 tokens 2048 x 1024
  // 3866 -> 3840.  a, b and the correction are read once, by streaming loads: the steps of 512 x 352 and 768 x 2048 0.7 to 1 % less, 2048 x
  // 1024 3808 -> 3790.  (Streaming stores of its results, of h and of the other GEMMs: within 0.5 % either way.)
  const int ds_c8 = lane % DS_CPR;
  const long ds_n = n0 + wn * (BN / 2) + ds_c8 * 8;
  const int ds_rows = (int)(m_end - m0);                        // valid rows of the tile
  const int ds_r0 = wm * (BM / 2) + lane / DS_CPR;
  const bool ds_nin = ds_n < Ndim;
  const unsigned ds_bytes = uniform((unsigned)(((long)(ds_rows - 1) * c_ms + Ndim) * 2)), ds_row_bytes = (unsigned)c_ms * 2;
  auto ds_rsrc = [&](const void* p, long elems, unsigned bytes) { return tile_rsrc(base_of(p, elems), bytes); };
  const long ds_tile = m0 * c_ms;
  __amdgpu_buffer_rsrc_t ds_in[3], ds_out[3];
  float ds_scale[BM > 128 ? 2 : 1];                             // of row `lane` of the wavefront's, and of the row 64 below
  if (EPI == kEpiDSwiglu) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      ds_in[i] = ds_rsrc(g.E[i], ds_tile, ds_bytes);
      ds_out[i] = ds_rsrc(g.C[i], ds_tile, ds_bytes);
    }
    const auto sc = ds_rsrc(g.row_scale, m0 * 2, (unsigned)ds_rows * 4u);
#pragma unroll
    for (int i = 0; i < (BM > 128 ? 2 : 1); ++i) ds_scale[i] = load4(sc, (unsigned)(wm * (BM / 2) + i * 64 + lane) * 4u);
  }
  auto ds_off = [&](int unit) {
    const int rt = ds_r0 + unit * DS_RPI;
    return rt < ds_rows && ds_nin ? (unsigned)rt * ds_row_bytes + (unsigned)ds_n * 2u : kOutOfRange;
  };
  rsrc_t ds_v[DS_AHEAD][3];
  if constexpr (EARLY) {
    // The first of these loads are spread over the last two iterations, in registers that the main loop has to spare.
    auto first_loads = [&](int n) { ds_v[n / 3][n % 3] = load16_once(ds_in[n % 3], ds_off(n / 3)); };
    constexpr int N2 = (2 * MF + EG - 1) / EG;             // by the next-to-last one
    static_assert(NSA == 3 && 2 * N2 >= DS_AHEAD * 3, "every K-tile and every one of these loads is requested");
    auto at_gap = [&](int q) { if (q % EG == 0 && q / EG < DS_AHEAD * 3) first_loads(q / EG); };
    step(std::integral_constant<int, kNextToLast>{}, at_gap);
    step(std::integral_constant<int, kLast>{}, [&](int q) { if (q % EG == 0 && N2 + q / EG < DS_AHEAD * 3) first_loads(N2 + q / EG); });
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(DS_AHEAD * 3) : "memory");      // no load may still write the LDS that the epilogue uses
  }
  // fp32 store epilogue: lanes along the columns, four of them per lane.  When the result is added to what is there,
  // the old values of a whole 32-row slab are requested before the previous slab is stored (loads and stores share one counter,
  // which counts them off in order: a load behind a store waits for that store, and one load, add, store chain per two rows would be
  // 64 round trips a tile; with the three matrices in one launch this took a step of gradient accumulation at 4096 tokens, 2048 x 2048, 8 of 32
  // experts from 1619 to 1471 us).  Only launches over operand sets add; the others keep neither the registers nor the code of it,
  // with which the down projection and the router GEMMs took 1 to 7 % longer (32768 tokens 4096 x 1408: 2955 -> 2923,
  // 77 -> 72 and 105 -> 102 us)
  constexpr int F_CPR = ECOLS / 4, F_RPI = 64 / F_CPR, F_NST = 32 / F_RPI;
  const long f_n = n0 + wn * (BN / 2) + (lane % F_CPR) * 4;
  float* const f_ct = reinterpret_cast<float*>(opC0) + e_tile;
  const bool f_add = SETS && g.accumulate;
  float4 f_old[SETS ? F_NST : 1];
  auto load_old = [&](int i) {
    if (SETS) {
#pragma unroll
      for (int st = 0; st < F_NST; ++st) {
        const int rt = e_r0 + i * 32 + st * F_RPI + lane / F_CPR;
        f_old[st] = *reinterpret_cast<const float4*>(
            f_ct + ((unsigned)(rt < e_rows ? rt : e_rows - 1) * (unsigned)c_ms + (unsigned)(f_n < Ndim ? f_n : 0)));
      }
    }
  };
  if (f_add) load_old(0);
  __syncthreads();                                   // the staging tiles are dead from here on
  rsrc_t ds_o[2][2];
  float* const ds_dots = reinterpret_cast<float*>(smem) + 4 * 32 * EPITCH + wave * (BM / 2);
#pragma unroll
  for (int i = 0; i < TS; ++i) {
    if (EPI == kEpiStore && !F32_OUT) {
      // bf16 output: round first, so that half as many bytes make the trip through LDS; rows of ECOLS bf16 with a
      // pitch of ECOLS*2+8 bytes (the 32 rows one write instruction touches fall into different banks)
      constexpr int BPITCH = ECOLS * 2 + 8;
      char* eb = reinterpret_cast<char*>(ep);
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
          *reinterpret_cast<uint2*>(eb + (ii * 16 + l16) * BPITCH + (j * 16 + lq * 4) * 2) =
              make_uint2(pack2(acc[j][2 * i + ii][0], acc[j][2 * i + ii][1]), pack2(acc[j][2 * i + ii][2], acc[j][2 * i + ii][3]));
      constexpr int CPR = ECOLS / 8, RPI = 64 / CPR;   // lanes per row (eight columns each), rows per access
      const int c8 = lane % CPR;
      const long n = n0 + wn * (BN / 2) + c8 * 8;
      const bool n_in = n < Ndim;
      bf16_t* ct = reinterpret_cast<bf16_t*>(opC0) + e_tile;
#pragma unroll
      for (int st = 0; st < 32 / RPI; ++st) {
        const int row = st * RPI + lane / CPR;
        const uint2 lo = *reinterpret_cast<const uint2*>(eb + row * BPITCH + c8 * 16);
        const uint2 hi = *reinterpret_cast<const uint2*>(eb + row * BPITCH + c8 * 16 + 8);
        const int rt = e_r0 + i * 32 + row;
        if (rt < e_rows && n_in)
          *reinterpret_cast<uint4*>(ct + ((unsigned)rt * (unsigned)c_ms + (unsigned)n)) = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
      continue;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int ii = 0; ii < 2; ++ii) {
        // The lane holds the 4-column group j*4 + lq of row ii*16 + l16.  The dSwiGLU epilogue reads two adjacent
        // groups per lane: even groups are kept in the first half of the LDS row and odd groups in the second, so that
        // each of its reads is contiguous across the lanes (the SwiGLU epilogue does the same inside the gate half
        // and inside the up half of its row: tiles j < TN/2 are the gate columns, the others the up columns)
        const int col = (EPI == kEpiDSwiglu) ? (lq & 1) * (ECOLS / 2) + (j * 2 + (lq >> 1)) * 4
                      : (EPI == kEpiSwiglu)  ? (j / (TN / 2)) * (ECOLS / 2) + (lq & 1) * (ECOLS / 4) + ((j % (TN / 2)) * 2 + (lq >> 1)) * 4
                                             : j * 16 + lq * 4;
        *reinterpret_cast<float4*>(ep + (ii * 16 + l16) * EPITCH + col) =
            make_float4(acc[j][2 * i + ii][0], acc[j][2 * i + ii][1], acc[j][2 * i + ii][2], acc[j][2 * i + ii][3]);
      }
    if (EPI == kEpiStore) {
      const bool n_in = f_n < Ndim;
      if (SETS) {
        float4 out[F_NST];
#pragma unroll
        for (int st = 0; st < F_NST; ++st) {
          out[st] = *reinterpret_cast<const float4*>(ep + (st * F_RPI + lane / F_CPR) * EPITCH + (lane % F_CPR) * 4);
          if (f_add) { out[st].x += f_old[st].x; out[st].y += f_old[st].y; out[st].z += f_old[st].z; out[st].w += f_old[st].w; }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (f_add && i + 1 < TS) load_old(i + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int st = 0; st < F_NST; ++st) {
          const int rt = e_r0 + i * 32 + st * F_RPI + lane / F_CPR;
          if (rt < e_rows && n_in) *reinterpret_cast<float4*>(f_ct + ((unsigned)rt * (unsigned)c_ms + (unsigned)f_n)) = out[st];
        }
      } else {
        // results that nothing is ever added to: stored as they are read
#pragma unroll
        for (int st = 0; st < F_NST; ++st) {
          const int row = st * F_RPI + lane / F_CPR, rt = e_r0 + i * 32 + row;
          const float4 v = *reinterpret_cast<const float4*>(ep + row * EPITCH + (lane % F_CPR) * 4);
          if (rt < e_rows && n_in) *reinterpret_cast<float4*>(f_ct + ((unsigned)rt * (unsigned)c_ms + (unsigned)f_n)) = v;
        }
      }
    } else if (EPI == kEpiSwiglu) {
      // LDS columns [0, ECOLS/2) hold the gate projection, [ECOLS/2, ECOLS) the up projection of the same output columns,
      // each with its even 4-column groups first and its odd ones behind.  A lane takes eight output columns of a row
      // (16-byte bf16 stores); the two rows that one 16-lane phase of a read touches are eight rows apart, which is 32
      // banks with this pitch.
      static_assert(EPI != kEpiSwiglu || (TN == 8 && ECOLS == 128), "lane layout of the SwiGLU epilogue");
      const int c8 = lane & 7, rsel = lane >> 3;
      const long n = n0 + wn * (BN / 4) + c8 * 8;
      const bool n_in = n < Ndim;
      bf16_t* cat = reinterpret_cast<bf16_t*>(g.C[0]) + e_tile;
      bf16_t* cbt = reinterpret_cast<bf16_t*>(g.C[1]) + e_tile;
      bf16_t* cht = reinterpret_cast<bf16_t*>(g.C[2]) + e_tile;
      bf16_t* cdt = reinterpret_cast<bf16_t*>(g.C[3]) + e_tile;
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        const int row = (st >> 1) * 16 + (st & 1) * 4 + (rsel >> 1) + 8 * (rsel & 1);
        const float* rp = ep + row * EPITCH + c8 * 4;
        const float4 a0 = *reinterpret_cast<const float4*>(rp), a1 = *reinterpret_cast<const float4*>(rp + ECOLS / 4);
        const float4 b0 = *reinterpret_cast<const float4*>(rp + ECOLS / 2), b1 = *reinterpret_cast<const float4*>(rp + 3 * ECOLS / 4);
        const int rt = e_r0 + i * 32 + row;
        if (rt < e_rows && n_in) {
          const unsigned ci = (unsigned)rt * (unsigned)c_ms + (unsigned)n;
          const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w}, b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
          // The backward needs a and b only to bf16 accuracy, but h = SiLU(a) b nearly to fp32 accuracy (its gate
          // gradient is a difference of nearly equal sums when experts are near copies).  Saved are therefore a and b
          // rounded to bf16 and the bf16 value of what the rounded pair misses, h - SiLU(bf16 a) (bf16 b): h comes back
          // to about 2^-17 from six bytes per element instead of eight.  The miss is taken to first order in the two
          // rounding steps (the second-order term is below 2^-18 of h), which needs no second sigmoid.
          uint32_t ap[4], bp[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) { ap[e] = pack2(a[2 * e], a[2 * e + 1]); bp[e] = pack2(b[2 * e], b[2 * e + 1]); }
          float h[8], dl[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float sg = sigmoidf_(a[e]);
            const float sl = a[e] * sg;                               // SiLU(a)
            h[e] = sl * b[e];
            const float ar = __uint_as_float((e & 1) ? (ap[e >> 1] & 0xffff0000u) : (ap[e >> 1] << 16));
            const float br = __uint_as_float((e & 1) ? (bp[e >> 1] & 0xffff0000u) : (bp[e >> 1] << 16));
            const float dsl = sg + sl * (1.f - sg);                   // SiLU'(a)
            // (the second product is the one that is rounded: left to the compiler, that changed with the loop around it)
            dl[e] = fmaf(dsl * (a[e] - ar), br, sl * (b[e] - br));
          }
          // the saved values are next read by the backward pass: streaming stores (h, which the next GEMM reads, stays plain)
          store_stream(reinterpret_cast<uint4*>(cat + ci), make_uint4(ap[0], ap[1], ap[2], ap[3]));
          store_stream(reinterpret_cast<uint4*>(cbt + ci), make_uint4(bp[0], bp[1], bp[2], bp[3]));
          store_stream(reinterpret_cast<uint4*>(cdt + ci),
                       make_uint4(pack2(dl[0], dl[1]), pack2(dl[2], dl[3]), pack2(dl[4], dl[5]), pack2(dl[6], dl[7])));
          *reinterpret_cast<uint4*>(cht + ci) = make_uint4(pack2(h[0], h[1]), pack2(h[2], h[3]), pack2(h[4], h[5]), pack2(h[6], h[7]));
        }
      }
    } else {
      // Two elements of a lane at a time, and behind each pair one or two of the memory instructions of the row groups before and
      // behind: the path takes a wavefront's 1 KB in sixteen cycles, and a wavefront that issues several in a row stands still for the
      // other three's.
      constexpr int UPS = 32 / DS_RPI;              // row groups per slab
      float4 uu[2][2];
      float rs[2];
      auto read_u = [&](int v) {
        const float* const p = ep + (v * DS_RPI + lane / DS_CPR) * EPITCH + ds_c8 * 4;
        uu[v & 1][0] = *reinterpret_cast<const float4*>(p);
        uu[v & 1][1] = *reinterpret_cast<const float4*>(p + ECOLS / 2);
        const int row = (i * UPS + v) * DS_RPI;
        rs[v & 1] = lane_value_at(ds_scale[row / 64], (row % 64) * 4 + lane / DS_CPR * 4);
      };
      read_u(0);
#pragma unroll
      for (int v = 0; v < UPS; ++v) {
        const int unit = i * UPS + v, far = unit - 1 + DS_AHEAD;
        const rsrc_t av = ds_v[unit % DS_AHEAD][0], bv = ds_v[unit % DS_AHEAD][1], dv = ds_v[unit % DS_AHEAD][2];
        const unsigned off_far = ds_off(far), off_prev = ds_off(unit - 1);
        rsrc_t (&o)[2] = ds_o[unit & 1], (&po)[2] = ds_o[1 - (unit & 1)];
        float dot = 0.f, h[8];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
          float da[2], db[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float a = __uint_as_float(e ? av[e2] & 0xffff0000u : av[e2] << 16), b = __uint_as_float(e ? bv[e2] & 0xffff0000u : bv[e2] << 16);
            const float hc = __uint_as_float(e ? dv[e2] & 0xffff0000u : dv[e2] << 16);
            const float4 u4 = uu[v & 1][e2 / 2];
            const float u = (e2 & 1) ? (e ? u4.w : u4.z) : (e ? u4.y : u4.x);
            const float sg = sigmoidf_(a);
            const float as = a * sg;          // SiLU of the saved (bf16) gate projection
            h[2 * e2 + e] = as * b + hc;      // the forward's h: what the rounded pair gives plus the saved correction
            dot = fmaf(u, h[2 * e2 + e], dot);
            const float dh = rs[v & 1] * u;
            da[e] = dh * b * (sg + as * (1.f - sg));
            db[e] = dh * as;
          }
          o[0][e2] = pack2(da[0], da[1]); o[1][e2] = pack2(db[0], db[1]);
          __builtin_amdgcn_sched_barrier(0);
          if (e2 == 0 && v + 1 < UPS) read_u(v + 1);
          if (unit > 0) {
            if (e2 < 3 && far < DS_UNITS) ds_v[far % DS_AHEAD][e2] = load16_once(ds_in[e2], off_far);
            if (e2 == 1 || e2 == 3) store16(ds_out[e2 / 2], off_prev, po[e2 / 2]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        asm("" : "+v"(dot));                 // (computed by all lanes: else the compiler branches around it)
        // gate-gradient partial of this row over the wavefront's columns: the CPR lanes of a row sit side by side
        dot = lane_group_sum<DS_CPR>(ds_off(unit) == kOutOfRange ? 0.f : dot);
        if (ds_c8 == 0) ds_dots[unit * DS_RPI + lane / DS_CPR] = dot;
        if (ds_store2) {
          const float r = rs[v & 1];
          store16(ds_out[2], ds_off(unit), rsrc_t{pack2(r * h[0], r * h[1]), pack2(r * h[2], r * h[3]), pack2(r * h[4], r * h[5]), pack2(r * h[6], r * h[7])});
        }
      }
      if (i + 1 == TS) {
#pragma unroll
        for (int x = 0; x < 2; ++x) store16(ds_out[x], ds_off(DS_UNITS - 1), ds_o[(DS_UNITS - 1) & 1][x]);
        const auto rd = ds_rsrc(g.rowdot, ((g.rowdot_slot0 + nt * 2 + wn) * g.rowdot_stride + m0) * 2, (unsigned)ds_rows * 4u);
#pragma unroll
        for (int x = 0; x < BM / 2; x += 64)
          if (x + lane < BM / 2) store4(rd, (unsigned)(wm * (BM / 2) + x + lane) * 4u, ds_dots[x + lane]);
      }
    }
  }
}

// C: the tile; CH: the shorter tile of the experts' last rows, or C again.
// An expert's last full tile holds 128 rows on average, and beside a round of 256 of them a launch of a few thousand tokens has few
// others.  Last tiles of up to 128 rows are therefore half as high: 0.7 of a full one's time, because each is alone with its
// panel of the weights.  They come last, where they also shorten the round that is not full: 4096 tokens, 32 experts of 2048 x 2048,
// top-4, gradient accumulation 1302 -> 1271 us; 16384, 32 of 3584 x 4864, top-2 7561 -> 7291; 12000, 48 of 4096 x 640, top-2
// 1128 -> 1094; layers whose experts end in few such tiles within 1 %.  In the order of the experts, beside the full tiles
// whose weights they share, they take 0.6 of one, but a full tile ends the launch: 1295 and 7610 us.
template <int MODE, int EPI, bool A_KC, bool B_KC, bool SETS, typename C, typename CH>
__global__ __launch_bounds__(256, C::MINB) void gemm_mfma_kernel(const GemmArgs g) {
  __shared__ uint4 smem[lds_units<C>() > lds_units<CH>() ? lds_units<C>() : lds_units<CH>()];
  int all = MODE == kRaggedM ? scalar_load(g.n_tiles) : 0, full = C::BM != CH::BM ? scalar_load(g.n_full) : 0;
  if (MODE == kRaggedM) asm volatile("" : "+s"(all), "+s"(full));          // one round trip
  if constexpr (C::BM != CH::BM) {
    static_assert(MODE == kRaggedM && CH::BN == C::BN && CH::BM == plan::kHalfRows, "the table's short tiles, the same columns");
    // The table has the full tiles first; the last round of them is cut in two where plan::tiles_cut says so.  Steps: 700 tokens 4096 x 1408, 8 experts top-2 413 -> 335 us, 1200 tokens 1032 x 1000, 12 experts 248 -> 195, 500 tokens 2048 x
    // 1024, 8 experts 175 -> 147, 3777 tokens 1536 x 1280, 16 experts 298 -> 288, 9000 tokens 2048 x 1024, 8 experts top-1 457 -> 431; eight
    // others 1.00 to 1.07 faster, launches of many rounds within 0.5 %.  Results are the same on either height.  The blocks of either height are dealt to the XCDs by themselves.
    const unsigned gx = (unsigned)cdiv(g.Ndim - g.n_base, EPI == kEpiSwiglu ? C::BN / 2 : C::BN);
    const unsigned tall = (unsigned)full * gx, shorts = (unsigned)(all - full) * gx;
    const unsigned cut = plan::tiles_cut(tall, shorts), whole = tall - cut;
    const unsigned first_short = (whole + kXcds - 1) / kXcds * kXcds;
    if (blockIdx.x >= first_short) {
      const unsigned at = dealt(blockIdx.x - first_short, 2 * cut + shorts);
      if (at >= 2 * cut + shorts) return;
      const bool of_tall = at < 2 * cut;
      gemm_tile<MODE, EPI, A_KC, B_KC, SETS, CH>(g, smem, of_tall ? whole + at / 2 : at - 2 * cut, of_tall ? 0 : full, of_tall ? full : all - full,
                                                 of_tall ? (int)(at & 1) : 0);
      return;
    }
    const unsigned at = dealt(blockIdx.x, whole);
    if (at < whole) gemm_tile<MODE, EPI, A_KC, B_KC, SETS, C>(g, smem, at, 0, full);
  } else if constexpr (SETS) {
    // the sets stand side by side, see there
    const unsigned per_set = (unsigned)cdiv(g.Mdim, C::BM) * (unsigned)cdiv(g.Ndim, C::BN);
    if (g.set[blockIdx.x / per_set % 3u].a_gather) gemm_tile<MODE, EPI, A_KC, B_KC, SETS, C, 1>(g, smem, blockIdx.x, 0, all);
    else gemm_tile<MODE, EPI, A_KC, B_KC, SETS, C, 2>(g, smem, blockIdx.x, 0, all);
  } else if constexpr (MODE == kRaggedM) {
    const unsigned total = (unsigned)all * (unsigned)cdiv(g.Ndim - g.n_base, EPI == kEpiSwiglu ? C::BN / 2 : C::BN), at = dealt(blockIdx.x, total);
    if (at < total) gemm_tile<MODE, EPI, A_KC, B_KC, SETS, C>(g, smem, at, 0, all);
  } else {
    gemm_tile<MODE, EPI, A_KC, B_KC, SETS, C>(g, smem, blockIdx.x, 0, 0);
  }
}

// the full tile: 256 x 256 x 64, one block per CU (all 160 KB of LDS, 256 accumulators per lane in AGPRs)
typedef Cfg<256, 256, 3, 2, 1> Tile;

// narrow outputs (the router scores of many tokens: half the matrix work on padding), the half-full last column
// tile of a ragged-row GEMM, and launches of few tiles
typedef Cfg<256, 128, 3, 3, 1> TileNarrow;
// few output rows (the router's weight gradient over many tokens has M <= 64 of them), the fused SwiGLU on 128-row tiles
// (plan::row_tile), and the last rows of an expert beside the full tile
typedef Cfg<128, 256, 3, 3, 1> TileShort;
// two blocks per CU, so that one block's memory phases overlap the other's: the ragged-row GEMMs but the fused SwiGLU on 128-row tiles,
// weight gradients of few full tiles (plan::wgrad_small_tiles), and the router's
typedef Cfg<128, 128, 3, 2, 2> TileSmall;
// the last rows of an expert beside TileNarrow
typedef Cfg<128, 128, 3, 2, 1> TileNarrowShort;
// ragged-row GEMMs on 64-row tiles (plan::row_tile), two blocks per CU: experts of few routed rows, bound by the stream of
// their weights, and narrow models with few tiles, bound by prologue and epilogue
typedef Cfg<64, 256, 2, 2, 2> Rows64;
typedef Cfg<64, 128, 3, 3, 2> Rows64Narrow;
static_assert(Tile::BM == plan::kFullRows && TileShort::BM == plan::kHalfRows && TileSmall::BM == plan::kHalfRows && Rows64::BM == plan::kQuarterRows &&
              Tile::BN == plan::kFullCols && TileNarrow::BN == plan::kHalfCols && TileSmall::BN == plan::kHalfCols && Rows64Narrow::BN == plan::kHalfCols,
              "the tiles that the plan counts");

template <int MODE, int EPI, bool A_KC, bool B_KC, typename C = Tile, bool SETS = false, typename CH = C>
int launch(const GemmArgs& g, hipStream_t s) {
  static_assert(!SETS || (MODE == kGroupedK && !A_KC && !B_KC && C::BM == C::BN), "operand sets: K-strided, square tiles");
  if (EPI == kEpiStore && (g.c_f32 != 0) != f32_out(MODE)) return SPES_EINVAL;
  if (MODE == kRaggedM && (g.a_rows != nullptr) != (EPI != kEpiStore)) return SPES_EINVAL;
  // operands are addressed with 32-bit byte offsets from their base
  if (SETS) {
    if (g.npairs != 1 || g.n_sets != 3) return SPES_EINVAL;
    for (int i = 0; i < g.n_sets; ++i) {
      if (g.set[i].a_elems <= 0 || g.set[i].b_elems <= 0) return SPES_EINVAL;
      if (g.set[i].a_elems >= (1L << 31) || g.set[i].b_elems >= (1L << 31)) return SPES_ESHAPE;
    }
  } else {
    if (g.a_elems <= 0 || g.b_elems <= 0 || g.accumulate) return SPES_EINVAL;
    if (g.a_elems >= (1L << 31) || g.b_elems >= (1L << 31)) return SPES_ESHAPE;
  }
  const int bno = (EPI == kEpiSwiglu) ? C::BN / 2 : C::BN;
  const int gx = cdiv(g.Ndim - (MODE == kRaggedM ? g.n_base : 0), bno);
  long total = (MODE == kRaggedM) ? (long)g.max_tiles * gx : (long)g.n_groups * cdiv(g.Mdim, C::BM) * gx;
  if (SETS) total *= g.n_sets;
  if (total <= 0) return SPES_OK;
  total = (total + kXcds - 1) / kXcds * kXcds;
  if (C::BM != CH::BM) total += kXcds + plan::kRound / 2;       // two kinds of tiles: rounded up twice, and up to half a round of them cut in two
  hipLaunchKernelGGL((gemm_mfma_kernel<MODE, EPI, A_KC, B_KC, SETS, C, CH>), dim3((unsigned)total), dim3(256), 0, s, g);
  return hipGetLastError() == hipSuccess ? SPES_OK : SPES_EHIP;
}

}  // namespace

// kRaggedM on row tiles shorter than 256.  W: the fused SwiGLU (gate and up columns side by side), N: everything else
template <typename W, typename N>
static int launch_short(int epi, bool b_kcontig, const GemmArgs& g, hipStream_t s) {
  if (epi == kEpiSwiglu && b_kcontig) return launch<kRaggedM, kEpiSwiglu, true, true, W>(g, s);
  if (epi == kEpiStore && b_kcontig) return launch<kRaggedM, kEpiStore, true, true, N>(g, s);
  if (epi == kEpiStore && !b_kcontig) return launch<kRaggedM, kEpiStore, true, false, N>(g, s);
  if (epi == kEpiDSwiglu && !b_kcontig) return launch<kRaggedM, kEpiDSwiglu, true, false, N>(g, s);
  return SPES_EINVAL;
}

// kRaggedM on full-height tiles and, for the last rows of an expert, half-height ones
template <typename C, typename CH>
static int launch_mixed(int epi, bool b_kcontig, const GemmArgs& g, hipStream_t s) {
  if (epi == kEpiStore && b_kcontig) return launch<kRaggedM, kEpiStore, true, true, C, false, CH>(g, s);
  if (epi == kEpiStore && !b_kcontig) return launch<kRaggedM, kEpiStore, true, false, C, false, CH>(g, s);
  if (epi == kEpiDSwiglu && !b_kcontig) return launch<kRaggedM, kEpiDSwiglu, true, false, C, false, CH>(g, s);
  return SPES_EINVAL;
}

// bf16 operands only.  a_kcontig / b_kcontig: the contraction index is the fast memory axis of that operand.
int launch_gemm_mfma(int mode, int epi, bool a_kcontig, bool b_kcontig, const GemmArgs& g, hipStream_t s) {
  if (mode == kRaggedM) {
    if (!a_kcontig) return SPES_EINVAL;
    if (g.row_tile == TileShort::BM) return launch_short<TileShort, TileSmall>(epi, b_kcontig, g, s);
    if (g.row_tile == Rows64::BM) return launch_short<Rows64, Rows64Narrow>(epi, b_kcontig, g, s);
    if (g.row_tile != Tile::BM) return SPES_EINVAL;
    // A last column tile that is at most half full goes to a launch of its own on the half-width tile (which costs
    // 0.6 of a full one) instead of running a full-width tile on half-empty operands.
    const int tail = plan::column_tail(g.Ndim);
    if (epi != kEpiSwiglu && g.n_base == 0 && tail > 0) {
      GemmArgs head = g, rest = g;
      head.Ndim = g.Ndim - tail;
      head.est_tiles = 0;            // both parts keep the slot numbering of full-width tiles
      rest.n_base = g.Ndim - tail;
      rest.rowdot_slot0 = 2 * (head.Ndim / Tile::BN);
      const int rc = launch_gemm_mfma(mode, epi, a_kcontig, b_kcontig, head, s);
      return rc != SPES_OK ? rc : launch_mixed<TileNarrow, TileNarrowShort>(epi, b_kcontig, rest, s);
    }
    if (epi != kEpiSwiglu && g.n_base == 0 && plan::few_tiles_narrow(g.Ndim, g.est_tiles))
      return launch_mixed<TileNarrow, TileNarrowShort>(epi, b_kcontig, g, s);
    if (epi == kEpiSwiglu && b_kcontig) return launch<kRaggedM, kEpiSwiglu, true, true, Tile, false, TileShort>(g, s);
    return launch_mixed<Tile, TileShort>(epi, b_kcontig, g, s);
  }
  if (epi != kEpiStore) return SPES_EINVAL;
  if (a_kcontig && b_kcontig)
    // router scores: 256-row tiles read the weights least often, but up to some thousand tokens leave most CUs idle for the time of one
    // tall tile.  64-row ones relative to them over 90 shapes (512, 1536 and 4096 wide, 8, 32 and 64 experts): 0.47 to 1.00 up to
    // 4096 tokens, 0.58 to 0.91 at 6000 and 8192; from 12000 on 0.71 to 1.28, on either side of 1 at each width
    return g.Mdim <= 8192 ? launch<kGroupedK, kEpiStore, true, true, Rows64Narrow>(g, s)
                          : launch<kGroupedK, kEpiStore, true, true, TileNarrow>(g, s);
  if (!a_kcontig && !b_kcontig) {
    if (g.n_sets > 0) {
      const long n = (long)g.n_sets * g.n_groups, full = n * plan::tiles(g.Mdim, g.Ndim, Tile::BM, Tile::BN),
                 small = n * plan::tiles(g.Mdim, g.Ndim, TileSmall::BM, TileSmall::BN);
      if (plan::wgrad_small_tiles(full, small, g.mean_k, g.max_k)) return launch<kGroupedK, kEpiStore, false, false, TileSmall, true>(g, s);
      return launch<kGroupedK, kEpiStore, false, false, Tile, true>(g, s);
    }
    // router weight gradient: the small tile relative to the wider one over the same shapes 0.79 to 1.00 up to 16384 tokens, beyond 0.78 to
    // 0.91 at 512 wide and 0.99 to 1.06 at 1536 and 4096
    if (g.Mdim <= TileShort::BM && g.Kdim <= 16384) return launch<kGroupedK, kEpiStore, false, false, TileSmall>(g, s);
    if (g.Mdim <= TileShort::BM) return launch<kGroupedK, kEpiStore, false, false, TileShort>(g, s);
    return launch<kGroupedK, kEpiStore, false, false>(g, s);
  }
  return SPES_EINVAL;
}

}  // namespace spes
