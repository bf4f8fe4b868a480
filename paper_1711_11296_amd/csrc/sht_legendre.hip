// Meridional (Legendre) stage of the transform pair on the matrix cores.
//
// Analysis, Sec. 3.1 eq. cc-quad with the parity fold of App. B (eqs. B3,
// B4): for every zonal wavenumber m,
//     a_n^m = sum_{j < ceil(J/2)} P~_n^m(mu_j) * (S^m_j if n-m even, A^m_j if odd)
// where S and A already carry the quadrature weight.  With all fields side
// by side this is, per m and parity, a dense product
//     C[n][c] = P[n][j] * B_par[j][c],  c = 2*field + {re, im},
// which the kernels run on MFMA (v_mfma_f32_16x16x4_f32 for FP32 data,
// v_mfma_f64_16x16x4_f64 for FP64 data).
//
// Synthesis, Sec. 2 eq. iLT split by parity (App. B): per m,
//     S^m_j = sum_{n-m even} P~_n^m(mu_j) a_n^m,  A^m_j = sum_{n-m odd} ...
// i.e. the same table read transposed.
//
// Table layout: two copies per (level, m), each blocked in the order its
// kernel streams it (analysis: rows r = n - m padded to 128 by Kp columns j;
// synthesis: 128-latitude tiles by blocks of 32 natural rows; zero padding;
// see the kernels below).  The split-bfloat16 kernels read the same FP32
// copies.  Workspace layouts: see ws_col and ws_block (the analysis reads
// rows of both parities interleaved in column blocks, the synthesis writes
// one plane per parity).
//
// Work decomposition: a host-built list gives one tile per workgroup; it is
// ordered so that the tiles of one m, which share the same right-hand
// operand, land on the same XCD (workgroups are dealt to the 8 XCDs round
// robin), and so that every XCD gets the same amount of work.

#include <hip/hip_runtime.h>

#include <type_traits>

#include "sht_device.h"
#include "sht_internal.h"

namespace sht {

// ---------------------------------------------------------------------------
// analysis: C[n][c] = P[n][j] * B_par(n)[j][c]
// tile = 128 consecutive rows r = n - m (both parities) x BN = 16*NCB
// columns, 8 waves.  Wave w: parity p = w & 1, row quarter q = w >> 1; it
// owns the 16 rows r = 32 q + 2 i + p (one MFMA row block) and all NCB
// column blocks.
// The contraction runs over j in blocks of KB.  Lane (i, g) of a wave
// supplies the k values j = 4 kk + g (kk < KB/4) of its row.  The analysis
// copy of the table is blocked per (128-row tile, KB columns) and, inside a
// block, per wave and per 64-lane vector, so that each wave streams its
// operands with fully contiguous 1 KiB loads straight into registers.
// The right-hand operand (both parities of the workspace block) goes from
// memory straight into LDS (global_load_lds, 64 x 16 bytes per instruction),
// rows 2 k + parity of BN columns, in two stages: the fills of block kb + 1
// are issued between the k-steps of block kb, one barrier per block.  Any
// NCB works.  Measured (MI355X, FP32, T479 with 100 fields): two tiles of 7
// blocks 0.264 ms against 0.345 ms for the 13 tiles of one block that a
// power-of-two choice leaves; T959 with 64 fields (NCB = 8) 1.01 ms, 112
// TFLOP/s: the shader clock drops to 2.0-2.15 GHz under matrix and memory
// load together (2.35 GHz for the same products from LDS alone), and at that
// clock the matrix cores are ~90 % busy.
// ---------------------------------------------------------------------------
template <typename T, int NCB, bool GEN = false>
struct AnalysisShape {
  static constexpr int E = 16 / (int)sizeof(T);        // scalars per 16 bytes
  // contraction block; generated P~ in FP64 also takes 32 latitudes (there
  // is no table layout to match, and a block's recurrence and two barriers
  // then serve twice the products)
  static constexpr int KB = (sizeof(T) == 4 || GEN) ? 32 : 16;
  static constexpr int KQ = KB / 4;                    // k values per lane and block
  static constexpr int BN = 16 * NCB;
  static constexpr int AHEAD = sizeof(T) == 4 && NCB <= 8 && !GEN ? 2 : 1;
  static constexpr int STAGE = 2 * KB * BN;            // elements of one stage: rows 2 k + parity of BN columns
  static constexpr int NCHUNK = STAGE / (64 * E);      // 1 KiB fills per stage, dealt to the 8 waves
  static constexpr int NB = (NCHUNK + 7) / 8;
  static constexpr int CS = BN + 1;                    // staging pitch of the output
  static constexpr int PS = 128 * KB;                  // generated P~ of one block (GEN)
  static constexpr size_t lds_bytes(bool gen) {
    const size_t main = (size_t)(2 * STAGE + (gen ? PS : 0)) * sizeof(T);
    const size_t cst = (size_t)64 * CS * sizeof(T);
    return main > cst ? main : cst;
  }
};

// The columns of a tile are dealt to the MFMA column blocks so that a lane's
// values of E blocks (16 bytes) lie side by side in an LDS row and one read
// fetches them: blocks E h + e of the whole groups take the columns
// 16 E h + E i + e (lane i), a remaining pair the columns base + 2 i + e, a
// single block base + i.
template <typename T>
__host__ __device__ constexpr int tile_col(int ncb, int c, int i) {
  const int E = 16 / (int)sizeof(T), whole = ncb / E * E;
  if (c < whole) return c / E * 16 * E + E * i + c % E;
  if (E == 4 && c < whole + 2 && ncb - whole >= 2) return 16 * whole + 2 * i + (c - whole);
  return 16 * c + i;
}

// Lane i's values of all column blocks from one LDS row.
template <typename T, int NCB>
__device__ __forceinline__ void read_cols(const T* row, int i, T (&b)[NCB]) {
  typedef typename V16<T>::type V;
  constexpr int E = 16 / (int)sizeof(T), W = NCB / E * E;
#pragma unroll
  for (int h = 0; h < W; h += E) {
    const V x = *reinterpret_cast<const V*>(row + 16 * h + E * i);
#pragma unroll
    for (int e = 0; e < E; ++e) b[h + e] = x[e];
  }
  if constexpr (NCB - W >= 2) {
    typedef T T2 __attribute__((ext_vector_type(2)));
    const T2 x = *reinterpret_cast<const T2*>(row + 16 * W + 2 * i);
    b[W] = x[0];
    b[W + 1] = x[1];
  }
  if constexpr ((NCB - W) & 1) b[NCB - 1] = row[16 * (NCB - 1) + i];
}

// Swizzle of the generated analysis block [128 rows][KB latitudes]: element
// (row, lat) sits at row * KB + (lat ^ gen_swz(row)), so that the 32
// latitudes one store instruction writes and the rows 2 i + p of one read
// instruction fall on distinct banks.
template <int KB>
__device__ __forceinline__ int gen_swz(int row) {
  return (2 * ((row >> 1) & 15)) & (KB - 1);
}

// GEN: the table operand is generated in the kernel (see gen_rows16): per K
// block, wave w produces the 16 rows of group w of the tile (lane l <
// KB at latitude l) into an LDS block, and after a barrier each wave reads
// its rows' values from it into the registers the table path fills from
// memory.
// The seed values of block kb + 2 are fetched while block kb is multiplied;
// the generated block is written after the products (its previous contents
// were read into registers before the last barrier), read after the next
// barrier, and a second barrier guards it against the next block's writes.
// Waves per SIMD the analysis is compiled for.  The FP64 generated kernel with
// 8 column blocks fills the LDS, one workgroup per compute unit: it takes the
// registers of two.  The FP32 generated kernels with one and two column blocks
// are bound by the recurrence's latency: within 80 registers three workgroups
// share a compute unit instead of two (N = 960, 641 rows, 3 fields 175 -> 161
// us; N = 1365, 16 fields 412 -> 387 with two blocks, 9 spills and all).
template <typename T, int NCB, bool GEN>
constexpr int analysis_wpe() {
  return sizeof(T) == 8 && GEN && NCB > 4 ? 2 : sizeof(T) == 4 && GEN && NCB <= 2 ? 6 : 4;
}

template <typename T, int NCB, bool GEN, int NL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(analysis_wpe<T, NCB, GEN>()))) void k_legendre_analysis(const GemmArgsN<NL> g) {
  typedef typename Acc<T>::type AccT;
  typedef typename V16<T>::type V;
  using S = AnalysisShape<T, NCB, GEN>;
  constexpr int E = S::E, KB = S::KB, KQ = S::KQ, BN = S::BN;

  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* Bs = reinterpret_cast<T*>(smem_raw);          // [2 stage][KB][2 parity][BN]

  const Tile t = g.tiles[blockIdx.x];
  if (t.level < 0) return;
  const LevelDesc& L = g.lev[NL == 1 ? 0 : t.level];
  const int N = L.N, m = t.m;
  const int nm = N - m + 1;
  const int r0 = t.rb * 128;
  const int c0 = t.cb * BN;
  const int Kp = L.Kp;
  const long long Cp = L.Cp;
  const T* wsm = static_cast<const T*>(g.ws) + L.ws_off + m * L.wblk;  // region m of row block 0
  const long long wjb = L.wjb;

  const int tid = threadIdx.x;
  // wave-uniform values live in scalar registers
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int p = w & 1, q = w >> 1;
  const int li = lane & 15, lg = lane >> 4;
  const bool active = r0 + 32 * q + p < nm;
  // this wave's run of the blocked table (see the table layout above)
  const T* arow = GEN ? nullptr
                      : static_cast<const T*>(g.table) + g.tab_off[L.m_base + m] + (long long)t.rb * Kp * 128 +
                            w * 16 * KB + lane * E;
  T* Ps = Bs + 2 * S::STAGE;  // GEN: [128 rows][KB latitudes], swizzled (gen_swz)
  // GEN: wave w generates group w (rows 16 w .. 16 w + 15 of the tile), lane
  // l at latitude l % KB of each block (lanes l and l + KB compute and
  // store the same values, which keeps the code free of branches); the
  // group's recurrence coefficients are held in lanes for the whole tile
  const int ggrp = w, glat = lane & (KB - 1);
  const int gi = t.rb * 8 + ggrp;
  const bool gon = GEN && 16 * gi < nm;  // uniform across the wave
  const double* gseed = GEN ? g.seeds + g.seed_off[L.m_base + m] + (gon ? 2LL * gi * Kp : 0LL) : nullptr;
  double gcA = 0.0, gcB = 0.0;
  if constexpr (GEN) gen_coef(g.rec + g.rec_off[L.m_base + m], 16 * gi, nm, lane, gcA, gcB);
  double gmu[2] = {0.0, 0.0}, gx0[2] = {0.0, 0.0}, gx1[2] = {0.0, 0.0};
  auto gen_fetch = [&](int kb, int set) __attribute__((always_inline)) {
    if constexpr (GEN) {
      if (gon) {
        const int j = kb * KB + glat;
        gmu[set] = L.murow[j];
        gx0[set] = gseed[j];
        gx1[set] = gseed[Kp + j];  // (a zero row when 16 gi + 1 = n_m: the seed rows are padded)
      }
    }
  };
  auto gen_store = [&](int set) __attribute__((always_inline)) {
    if constexpr (GEN) {
      gen_rows16<false>(gcA, gcB, 16 * gi, nm, gmu[set], gx0[set], gx1[set], [&](int s2, double x) {
        const int row = 16 * ggrp + s2;
        Ps[row * KB + (glat ^ gen_swz<KB>(row))] = (T)x;
      });
    }
  };
  T areg[KQ];
  auto gen_read = [&]() __attribute__((always_inline)) {
    const int rr = 32 * q + 2 * li + p;
#pragma unroll
    for (int kk = 0; kk < KQ; ++kk) areg[kk] = Ps[rr * KB + ((4 * kk + lg) ^ gen_swz<KB>(rr))];
  };

  AccT acc[NCB];
#pragma unroll
  for (int c = 0; c < NCB; ++c) acc[c] = AccT{0, 0, 0, 0};

  // Both operands are fetched one K block ahead: the table's into two register
  // sets used in turn (loop unrolled by two), the workspace's into two LDS
  // stages.
  V an[2][KQ / E];
  // (issued unconditionally, also by waves without rows in this tile and
  // for blocks past the end, clamped: with straight-line loads the wait
  // counts cover exactly the block that is consumed)
  auto gload_a = [&](int kb, V (&av)[KQ / E]) {
#pragma unroll
    for (int v = 0; v < KQ / E; ++v) av[v] = *reinterpret_cast<const V*>(arow + kb * 128 * KB + v * 64 * E);
  };
  // memory -> LDS without registers: instruction i of wave w fills the
  // 1 KiB chunk number i*8 + w of the stage; lane l takes its 16-byte piece
  // (row 2 k + parity, physical column) and fetches the logical column under
  // the swizzle.  The lane's byte offsets within a K block are fixed for the
  // tile (32-bit, from the block's uniform base).
  // (with an odd number of chunk rows the last wave's chunk is filled by
  // several waves with the same values, which keeps the loop free of branches)
  auto chunk = [&](int i) __attribute__((always_inline)) {
    return S::NCHUNK % 8 == 0 ? i * 8 + w : min(i * 8 + w, S::NCHUNK - 1);
  };
  unsigned dofs[S::NB];
#pragma unroll
  for (int i = 0; i < S::NB; ++i) {
    const int u = chunk(i) * 64 + lane;
    const int rr = u / (BN / E), col = (u - rr * (BN / E)) * E;
    const int k = rr >> 1, par = rr & 1;
    dofs[i] = (unsigned)(k * 2 * (int)Cp + ws_col(L.wsh, par, c0 + col)) * (unsigned)sizeof(T);
  }
  auto dma1 = [&](int i, int kb, int stage) __attribute__((always_inline)) {
    // K block kb: rows KB kb .. of row block KB kb / 32
    const long long ko = KB == SHT_K_PAD ? kb * wjb : (kb >> 1) * wjb + (kb & 1) * (KB * 2 * Cp);
    load_to_lds16(reinterpret_cast<const char*>(wsm + ko) + dofs[i],
                  Bs + stage * S::STAGE + chunk(i) * 64 * E);
  };
  auto dma = [&](int kb, int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < S::NB; ++i) dma1(i, kb, stage);
  };
  // Wait for this wave's LDS fills (and table loads): both are issued at the
  // start of a block and wanted at its end.  Only a wait for all of them is
  // safe: fills into LDS and loads into registers complete out of order
  // with respect to each other (a wait for all but the two table loads
  // issued after the fills let a barrier pass with fills in flight).
  auto wait_fills = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_vm(0));
  };
  // one K block's products; the fills of the next block are issued between
  // the k-steps
  auto compute = [&](int stage, const V (&av)[KQ / E], int kn) __attribute__((always_inline)) {
    const T* Bp = Bs + stage * S::STAGE + (2 * lg + p) * BN;
    // the reads of a k-step are issued AH steps ahead of its products
    constexpr int AH = S::AHEAD;
    T bv[AH + 1][NCB];
#pragma unroll
    for (int kk = 0; kk < AH; ++kk) read_cols<T, NCB>(Bp + 8 * kk * BN, li, bv[kk]);
#pragma unroll
    for (int kk = 0; kk < KQ; ++kk) {
      T a;
      if constexpr (GEN) a = areg[kk];
      else a = av[kk / E][kk % E];
      if (kk + AH < KQ) read_cols<T, NCB>(Bp + 8 * (kk + AH) * BN, li, bv[(kk + AH) % (AH + 1)]);
      if (kk < S::NB) dma1(kk, kn, 1 - stage);
#pragma unroll
      for (int c = 0; c < NCB; ++c) acc[c] = mfma16(a, bv[kk % (AH + 1)][c], acc[c]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = KQ; i < S::NB; ++i) dma1(i, kn, 1 - stage);
  };
  const int nkb = Kp / KB;
  // one K block; H = kb & 1 selects the table registers of block kb (and of
  // kb + 2), 1 - H those of block kb + 1
  auto step = [&](auto hc, auto on, int kb) __attribute__((always_inline)) {
    constexpr int H = decltype(hc)::value;
    // after the last block the idle stage receives a clamped block that
    // nothing reads, which keeps the loop free of branches around memory
    // operations
    const int kn = kb + 1 < nkb ? kb + 1 : nkb - 1;
    gen_fetch(kb + 2 < nkb ? kb + 2 : nkb - 1, H);
    if constexpr (!GEN) gload_a(kn, an[1 - H]);
    if constexpr (decltype(on)::value)
      compute(H, an[H], kn);
    else
      dma(kn, 1 - H);
    gen_store(1 - H);  // block kb + 1 (clamped after the last: nothing reads it)
    wait_fills();
    lds_barrier();
    if constexpr (GEN) {
      gen_read();
      lds_barrier();
    }
  };
  auto kloop = [&](auto on, int kb) __attribute__((always_inline)) {
    for (; kb + 1 < nkb; kb += 2) {
      step(std::integral_constant<int, 0>{}, on, kb);
      step(std::integral_constant<int, 1>{}, on, kb + 1);
    }
    if (kb < nkb) step(std::integral_constant<int, 0>{}, on, kb);
  };

  // reduced transform: the blocks before kb0 hold only latitudes where
  // every |P~_n^m| < 1e-16 (kb0 = 0 otherwise)
  const int kb0 = min(g.jstart[L.m_base + m] / KB, nkb - 1);
  dma(kb0, 0);
  asm volatile("" ::: "memory");
  if constexpr (GEN) {
    gen_fetch(kb0, 0);
    gen_store(0);
    gen_fetch(kb0 + 1 < nkb ? kb0 + 1 : nkb - 1, 1);
  } else {
    gload_a(kb0, an[0]);
  }
  __builtin_amdgcn_s_waitcnt(wait_vm(0));
  __syncthreads();
  if constexpr (GEN) {
    gen_read();
    __syncthreads();
  }
  // waves without rows in this tile run the loop without products
  if (active)
    kloop(std::true_type{}, kb0);
  else
    kloop(std::false_type{}, kb0);

  // stage 64 rows at a time in LDS, then write spec rows contiguously
  T* Cs = Bs;  // [64][CS]
  T* spec = static_cast<T*>(g.spec_out) + L.spec_off;
  const long long nc = (long long)(N + 1) * (N + 2) / 2;
  const long long base = spec_idx(N, m, m);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if ((q >> 1) == h) {
#pragma unroll
      for (int c = 0; c < NCB; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int rl = 32 * (q & 1) + 2 * out_row<T>(lg, i) + p;
          Cs[rl * S::CS + tile_col<T>(NCB, c, li)] = acc[c][i];
        }
    }
    __syncthreads();
    for (int qq = tid; qq < 64 * (BN / 2); qq += 512) {
      const int fl = qq >> 6, rl = qq & 63;
      const int f = (c0 >> 1) + fl;
      const int r = r0 + 64 * h + rl;
      if (r < nm && f < L.F) {
        T* d = spec + ((long long)f * nc + base + r) * 2;
        d[0] = Cs[rl * S::CS + 2 * fl];
        d[1] = Cs[rl * S::CS + 2 * fl + 1];
      }
    }
    if (h == 0) __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// synthesis: S_p[j][c] = sum_{r of parity p} P[r][j] * a[r][c]
// tile = 128 latitudes j x BN = 16*NCB columns, both parities, 8 waves.
// Wave w: parity p = w & 1, latitude quarter q = w >> 1; it owns the 32
// latitudes j = 32 q + 16 jb + i (jb < 2, two MFMA row blocks) and all NCB
// column blocks.  The contraction runs over r' (r = 2 r' + p) in blocks of
// KR per parity; lane (i, g) supplies r' = g KR/4 + kk (kk < KR/4).
// The table operand comes straight from memory into registers: the
// synthesis copy is blocked per (m, 128-latitude tile, K block), inside a
// block per wave and per 64-lane vector (vector v of lane (i, g) holds
// latitude block jb = v / (KQ/E) and r' = g KQ + E (v % (KQ/E)) + e).
// The spectral operand goes through LDS in two stages, transposed to
// [parity][column][r'] so that each lane reads its KR/4 values of a column
// as 16-byte vectors; one barrier per block.
// ---------------------------------------------------------------------------
template <typename T, int NCB>
struct SynthesisShape {
  static constexpr int E = 16 / (int)sizeof(T);
  static constexpr int KR = 16;                         // r' per parity and block
  static constexpr int KQ = KR / 4;                    // r' per lane and block
  static constexpr int BN = 16 * NCB;
  static constexpr int PITCH = KR + 16 / (int)sizeof(T);  // 16-byte pad: 4 mod 32 words
  static constexpr int STAGE = 2 * BN * PITCH;
  static constexpr int NV = 2 * KQ / E;                // table vectors per lane and block
  static constexpr int QUADS = (BN / 2) * (KR / 2);    // 4 natural rows of one field
  static constexpr int NQ = (QUADS + 511) / 512;
  static constexpr int CHUNK = 128 * 2 * KR;           // table elements per block
  static constexpr int GP = 130;                       // GEN: pitch of the generated block [2 KR rows][128 latitudes]
  static constexpr size_t lds_bytes(bool gen) { return (size_t)(2 * STAGE + (gen ? 2 * KR * GP : 0)) * sizeof(T); }
};

// GEN: the table operand is generated in the kernel (see gen_rows16): per K
// block of 2 KR natural rows (two 16-degree groups), waves 0..3 produce the
// 16 rows of one group for 64 latitudes of the tile each into an LDS block
// [row][latitude] (pitch 130: the reads of one instruction, 16 latitudes by
// 4 rows, fall on distinct banks); barriers as in the analysis.
template <typename T, int NCB, bool GEN, int NL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2))) void k_legendre_synthesis(const GemmArgsN<NL> g) {
  typedef typename Acc<T>::type AccT;
  typedef typename V16<T>::type V;
  using S = SynthesisShape<T, NCB>;
  constexpr int E = S::E, KR = S::KR, KQ = S::KQ, BN = S::BN, PITCH = S::PITCH;

  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* Bs = reinterpret_cast<T*>(smem_raw);  // [2 stage][2 parity][BN][PITCH]

  const Tile t = g.tiles[blockIdx.x];
  if (t.level < 0) return;
  const LevelDesc& L = g.lev[NL == 1 ? 0 : t.level];
  const int N = L.N, m = t.m;
  const int nm = N - m + 1;
  const int nkb = (nm + 2 * KR - 1) / (2 * KR);
  const int jt = t.rb;
  const int c0 = t.cb * BN;
  const long long Cp = L.Cp;
  const T* spec = static_cast<const T*>(g.spec_in) + L.spec_off;
  const long long nc = (long long)(N + 1) * (N + 2) / 2;
  const long long sbase = spec_idx(N, m, m);

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int p = w & 1, q = w >> 1;
  const int li = lane & 15, lg = lane >> 4;
  const bool active = jt * 128 + 32 * q < L.Jh;
  const T* arun = GEN ? nullptr
                      : static_cast<const T*>(g.table) + g.tab_off[L.m_base + m] + (long long)jt * nkb * S::CHUNK +
                            w * (S::CHUNK / 8) + lane * E;
  T* Ps = Bs + 2 * S::STAGE;  // GEN: [2 KR rows][GP]
  // GEN: waves 0..3 generate; wave w takes group gsub = w >> 1 of each block
  // (rows 16 gsub .. + 15 of the block, uniform across the wave) at
  // latitude glat = 64 (w & 1) + lane of the tile; the group's recurrence
  // coefficients are fetched into lanes with its seed values
  const int gsub = w >> 1, glat = 64 * (w & 1) + lane;
  const int gj = jt * 128 + glat;
  const bool gthr = GEN && w < 4;  // uniform across the wave
  const bool gjin = gthr && gj < L.Kp;
  const double* gseeds = GEN ? g.seeds + g.seed_off[L.m_base + m] : nullptr;
  const double* grec = GEN ? g.rec + g.rec_off[L.m_base + m] : nullptr;
  const double gmu = (GEN && gjin) ? L.murow[gj] : 0.0;
  double gx0[2] = {0.0, 0.0}, gx1[2] = {0.0, 0.0}, gcA[2] = {0.0, 0.0}, gcB[2] = {0.0, 0.0};
  auto gen_fetch = [&](int kb, int set) __attribute__((always_inline)) {
    if constexpr (GEN) {
      const int gi = 2 * kb + gsub;
      if (gthr) gen_coef(grec, 16 * gi, nm, lane, gcA[set], gcB[set]);
      if (gjin && 16 * gi < nm) {
        gx0[set] = gseeds[2LL * gi * L.Kp + gj];
        gx1[set] = gseeds[(2LL * gi + 1) * L.Kp + gj];  // zero row when 16 gi + 1 = n_m
      }
    }
  };
  auto gen_store = [&](int kb, int set) __attribute__((always_inline)) {
    if constexpr (GEN) {
      if (gthr) {
        const int gi = 2 * kb + gsub;
        gen_rows16<false>(gcA[set], gcB[set], 16 * gi, gjin ? nm : 0, gmu, gx0[set], gx1[set],
                          [&](int s2, double x) { Ps[(16 * gsub + s2) * S::GP + glat] = (T)x; });
      }
    }
  };
  T areg[2][KQ];
  auto gen_read = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
      for (int kk = 0; kk < KQ; ++kk) areg[jb][kk] = Ps[(2 * (lg * KQ + kk) + p) * S::GP + 32 * q + 16 * jb + li];
  };

  AccT acc[2][NCB];
#pragma unroll
  for (int jb = 0; jb < 2; ++jb)
#pragma unroll
    for (int c = 0; c < NCB; ++c) acc[jb][c] = AccT{0, 0, 0, 0};

  constexpr int QV = 8 / E;  // vectors per quad: 4 rows (re, im) of one field
  // Operands are fetched two K blocks ahead into two register sets used in
  // turn (the loop is unrolled by two so that the set is a compile-time
  // choice): block kb + 2 is requested while block kb is multiplied, and
  // block kb + 1, requested one block earlier, goes to LDS afterwards.
  V an[2][S::NV], ac[S::NV];
  V rq[2][S::NQ][QV];
  // The tile's spectra as a buffer starting at its first field and wave
  // number: reads past the end of the level's spectra return zero (fields
  // beyond F), rows beyond n = N are masked; offsets stay below 4 GiB (at
  // most 16 NCB fields of at most (N+1)(N+2)/2 rows).
  const long long sfirst = ((long long)(c0 >> 1) * nc + sbase) * 2;
  long long sbytes = ((long long)L.F * nc * 2 - sfirst) * (long long)sizeof(T);
  if (sbytes < 0) sbytes = 0;  // a tile past the last field (all its reads are zeros)
  const __amdgpu_buffer_rsrc_t srs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>(spec + sfirst), (short)0, (int)(unsigned)(sbytes > 0xFFFFFFFFLL ? 0xFFFFFFFFLL : sbytes),
      0x00020000);
  // Quad task qq: field fl, quad rp (natural rows 4 rp .. 4 rp + 3 of the
  // block).  In the FP32 form the lanes of a half-wave take 4 quads of 8
  // fields, so that the 8-byte stores of one instruction (column 2 fl + ri,
  // pitch 20 words) cover all 64 LDS banks once; otherwise quads vary
  // fastest.
  auto quad_of = [&](int qq, int& fl, int& rp) __attribute__((always_inline)) {
    if constexpr (sizeof(T) == 4 && KR / 2 == 8) {
      rp = (qq & 3) | (((qq >> 5) & 1) << 2);
      fl = ((qq >> 2) & 7) | ((qq >> 6) << 3);
    } else {
      fl = qq / (KR / 2);
      rp = qq % (KR / 2);
    }
  };
  // (issued unconditionally, also by waves without latitudes in this tile
  // and for blocks past the end, clamped: with straight-line loads the
  // compiler's wait counts cover exactly the block that is consumed)
  auto gload = [&](int kb, V (&av)[S::NV], V (&bq)[S::NQ][QV]) {
    if constexpr (!GEN) {
#pragma unroll
      for (int v = 0; v < S::NV; ++v)
        av[v] = *reinterpret_cast<const V*>(arun + (long long)kb * S::CHUNK + v * 64 * E);
    }
#pragma unroll
    for (int i = 0; i < S::NQ; ++i) {
      const int qq = tid + i * 512;
      int fl, rp;
      quad_of(qq, fl, rp);
      const int r = kb * 2 * KR + 4 * rp;  // first natural row of the quad
      const unsigned off = ((unsigned)fl * (unsigned)nc + (unsigned)r) * 2u * (unsigned)sizeof(T);
      // vector u holds natural rows r + u E/2 .. r + (u+1) E/2 - 1; rows
      // beyond n = N are masked when the quad is stored to LDS
#pragma unroll
      for (int u = 0; u < QV; ++u)
        bq[i][u] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(srs, (int)(off + 16u * u), 0, 0));
    }
  };
  auto lstore = [&](int stage, const V (&bq)[S::NQ][QV], int kb) {
    T* dst = Bs + stage * S::STAGE;
#pragma unroll
    for (int i = 0; i < S::NQ; ++i) {
      const int qq = tid + i * 512;
      if (S::NQ * 512 == S::QUADS || qq < S::QUADS) {
        int fl, rp;
        quad_of(qq, fl, rp);
        const int r = kb * 2 * KR + 4 * rp;
        T x[8];
#pragma unroll
        for (int u = 0; u < QV; ++u)
#pragma unroll
          for (int e = 0; e < E; ++e) x[u * E + e] = r + (u * E + e) / 2 < nm ? bq[i][u][e] : (T)0;
        // x = re, im of natural rows r, r+1, r+2, r+3: parity par, r' = 2 rp + h
#pragma unroll
        for (int par = 0; par < 2; ++par)
#pragma unroll
          for (int ri = 0; ri < 2; ++ri) {
            typedef T T2 __attribute__((ext_vector_type(2)));
            *reinterpret_cast<T2*>(dst + (par * BN + 2 * fl + ri) * PITCH + 2 * rp) =
                T2{x[2 * par + ri], x[4 + 2 * par + ri]};
          }
      }
    }
  };
  auto compute = [&](int stage) {
    T a[2][KQ];
    if constexpr (GEN) {
#pragma unroll
      for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) a[jb][kk] = areg[jb][kk];
    } else {
#pragma unroll
      for (int v = 0; v < S::NV; ++v)
#pragma unroll
        for (int e = 0; e < E; ++e) a[v / (KQ / E)][(v % (KQ / E)) * E + e] = ac[v][e];
    }
    const T* Bp = Bs + stage * S::STAGE + (p * BN + li) * PITCH + lg * KQ;
#pragma unroll
    for (int c = 0; c < NCB; ++c) {
      T bv[KQ];
#pragma unroll
      for (int v = 0; v < KQ / E; ++v) {
        const V x = *reinterpret_cast<const V*>(Bp + c * 16 * PITCH + v * E);
#pragma unroll
        for (int e = 0; e < E; ++e) bv[v * E + e] = x[e];
      }
#pragma unroll
      for (int kk = 0; kk < KQ; ++kk)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) acc[jb][c] = mfma16(a[jb][kk], bv[kk], acc[jb][c]);
    }
    // the reads of a column block are issued two column blocks ahead
    constexpr int RDC = KQ / E;
    mfma_lds_pipeline<2 * RDC, (NCB - 2) * RDC, (2 * KQ + RDC - 1) / RDC, 4 * KQ>();
  };
  // one K block; H = kb & 1 selects the register set of block kb (and of
  // kb + 2), 1 - H that of block kb + 1
  auto step = [&](auto hc, int kb) {
    constexpr int H = decltype(hc)::value;
    gen_fetch(kb + 2 < nkb ? kb + 2 : nkb - 1, H);
    gload(kb + 2 < nkb ? kb + 2 : nkb - 1, an[H], rq[H]);
    if (active) compute(H);
    // after the last block this fills the idle stage with a clamped block
    // (nothing reads it), which keeps the loop free of branches around
    // memory operations
    lstore(1 - H, rq[1 - H], kb + 1 < nkb ? kb + 1 : nkb - 1);
    gen_store(kb + 1 < nkb ? kb + 1 : nkb - 1, 1 - H);
    if constexpr (!GEN) {
#pragma unroll
      for (int v = 0; v < S::NV; ++v) ac[v] = an[1 - H][v];
    }
    lds_barrier();
    if constexpr (GEN) {
      gen_read();
      lds_barrier();
    }
  };

  // reduced transform: a tile whose latitudes all lie below the first one
  // kept for this m writes zeros (uniform across the workgroup)
  if (jt * 128 + 128 > g.jstart[L.m_base + m]) {
    gload(0, an[0], rq[0]);
    gload(nkb > 1 ? 1 : 0, an[1], rq[1]);
    lstore(0, rq[0], 0);
    if constexpr (GEN) {
      gen_fetch(0, 0);
      gen_store(0, 0);
      gen_fetch(nkb > 1 ? 1 : 0, 1);
    } else {
#pragma unroll
      for (int v = 0; v < S::NV; ++v) ac[v] = an[0][v];
    }
    __syncthreads();
    if constexpr (GEN) {
      gen_read();
      __syncthreads();
    }
    for (int kb = 0; kb < nkb; kb += 2) {
      step(std::integral_constant<int, 0>{}, kb);
      if (kb + 1 < nkb) step(std::integral_constant<int, 1>{}, kb + 1);
    }
  }

  if (!active) return;
  // the wave's 32 latitudes are one row block
  const int jblk = jt * 4 + q;
  T* ws = static_cast<T*>(g.ws) + L.ws_off + jblk * L.wjb + m * L.wblk + p * ws_odd(L.Jh, Cp, L.wblk, jblk);
#pragma unroll
  for (int jb = 0; jb < 2; ++jb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = jt * 128 + 32 * q + 16 * jb + out_row<T>(lg, i);
      if (j < L.Jh) {
#pragma unroll
        for (int c = 0; c < NCB; ++c) ws[(j % SHT_K_PAD) * Cp + c0 + c * 16 + li] = acc[jb][c][i];
      }
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
constexpr int kMaxSynthesisNcb = 8;

template <typename T, int NCB, bool GEN, int NL>
static hipError_t launch_ncb(bool analysis, const GemmArgsN<NL>& g, hipStream_t st) {
  const dim3 grid(g.ntiles), block(512);
  if constexpr (sizeof(T) == 8 && NCB > 8) return hipErrorInvalidValue;  // FP64 takes at most 8
  else if (analysis) {
    // (widths that would spill: tile_spills never lets a plan choose them)
    if constexpr (sizeof(T) == 4 && GEN && (NCB == 7 || NCB == 9)) return hipErrorInvalidValue;
    else {
      const size_t lds = AnalysisShape<T, NCB, GEN>::lds_bytes(GEN);
      lds_optin<k_legendre_analysis<T, NCB, GEN, NL>>(lds);
      hipLaunchKernelGGL((k_legendre_analysis<T, NCB, GEN, NL>), grid, block, lds, st, g);
    }
  } else {
    // wider synthesis tiles do not fit the register file
    if constexpr (NCB > kMaxSynthesisNcb) return hipErrorInvalidValue;
    else {
      const size_t lds = SynthesisShape<T, NCB>::lds_bytes(GEN);
      lds_optin<k_legendre_synthesis<T, NCB, GEN, NL>>(lds);
      hipLaunchKernelGGL((k_legendre_synthesis<T, NCB, GEN, NL>), grid, block, lds, st, g);
    }
  }
  return hipGetLastError();
}

template <typename T, bool GEN, int NL>
static hipError_t launch_legendre_t(bool analysis, const GemmArgsN<NL>& g, int ncb, hipStream_t st) {
  switch (ncb) {
    case 1: return launch_ncb<T, 1, GEN>(analysis, g, st);
    case 2: return launch_ncb<T, 2, GEN>(analysis, g, st);
    case 3: return launch_ncb<T, 3, GEN>(analysis, g, st);
    case 4: return launch_ncb<T, 4, GEN>(analysis, g, st);
    case 5: return launch_ncb<T, 5, GEN>(analysis, g, st);
    case 6: return launch_ncb<T, 6, GEN>(analysis, g, st);
    case 7: return launch_ncb<T, 7, GEN>(analysis, g, st);
    case 8: return launch_ncb<T, 8, GEN>(analysis, g, st);
    case 9: return launch_ncb<T, 9, GEN>(analysis, g, st);
    case 10: return launch_ncb<T, 10, GEN>(analysis, g, st);
    default: return hipErrorInvalidValue;
  }
}

template <int NL>
static hipError_t launch_legendre_n(int form, bool analysis, const GemmArgsN<NL>& g, int ncb, bool gen,
                                    hipStream_t st) {
  if (form == SHT_FORM_FP64)
    return gen ? launch_legendre_t<double, true>(analysis, g, ncb, st)
               : launch_legendre_t<double, false>(analysis, g, ncb, st);
  return gen ? launch_legendre_t<float, true>(analysis, g, ncb, st)
             : launch_legendre_t<float, false>(analysis, g, ncb, st);
}

int launch_legendre(int form, bool analysis, const GemmArgs& g, int ncb, bool gen, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (g.ntiles <= 0) return (int)hipSuccess;
  if (form == SHT_FORM_BF16X6) return (int)launch_legendre_bf16(analysis, g, ncb, gen, st);
  return (int)(g.nlev == 1 ? launch_legendre_n(form, analysis, one_level(g), ncb, gen, st)
                           : launch_legendre_n(form, analysis, g, ncb, gen, st));
}

}  // namespace sht
