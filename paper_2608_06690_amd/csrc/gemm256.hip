// Grouped bf16 GEMM on 256 x 256 output tiles with K steps of 64: the prefill and training
// products of the experts (and of the always-on shared group).
//
//   GEMM1  [rows, H] x [H, 2I]: a tile holds 128 gate and the matching 128 up columns, so
//          h = silu(g) * u is formed in registers and rounded once to bf16;
//   GEMM2  [rows, I] x [I, H] -> y_perm; the first N tile of each private M tile adds its
//          rows to the execution audit;
//   plain  GEMM2 without the audit, its A rows read in place or gathered by token (the
//          backward's products with transposed weights).
//
// Tile list: groups are the routed experts and the shared group; a tile is (group, M tile of
// 256 rows, N tile). Every block scans the per-group tile counts on the device, so groups
// without rows get no tile and load nothing.
//
// Schedule. 8 waves as 2 row groups x 4 column groups, two waves per SIMD (one of each row
// group). A K step's operands are four half tiles of 128 rows x 128 bytes (A0, A1, B0, B1), and
// a wave owns a 64 x 32 block of each of the four (A half, B half) quadrants. A step is four
// phases, one quadrant each; a phase reads the half tiles it needs into registers, issues the
// global->LDS copies of the half tiles two steps ahead whose slots the previous phase freed,
// and multiplies. The row groups run one half phase apart (two barriers per phase), so on each
// SIMD one wave multiplies while the other reads and copies. A half tile is overwritten as
// soon as it has been read, not when its step ends, so 80-96 KiB of copies stay in flight per
// CU across step and tile boundaries: waits count the younger copies and never drain the queue.
// Tiles of up to 128 rows have no A1: two phases per step, a quarter fewer copies and half the
// MFMAs. A last half with few valid rows (the usual one where experts have ragged counts)
// multiplies its 16-row blocks up to the last valid one, by bodies of up to 32 and 64 rows of a
// second half, whose two quadrants then share a phase, and of up to 64 rows of a first one. With
// whole halves only, tiles of 129 to 192 rows cost what 256 rows cost, more than kernels that
// skip such blocks: 144 rows drawn per expert over 48 experts of 1152 x 704 98 us, 80 with these
// bodies; 160 of 2048 x 768 406, 366; 320 rows over 16 of 7168 x 2048 628, 607.
//
// The weight fragment is the first MFMA operand, and the weight rows of a 32-row block are
// permuted in LDS, so that a lane's results are 8 consecutive output columns of one row: the
// epilogue goes from the accumulators to 16-byte stores without LDS or barriers.
//
// What bounds it: the global->LDS copies. Measured per call of the two forward products (MI355X;
// timing builds before the short last halves): 16384 tokens over 32 experts 1,202 us, copies alone
// 913, MFMAs and LDS reads alone 767; 4096 tokens over 160 experts 493, 415 and 317. 46 to 68
// lines per CU are on their way from L2 whatever is issued ahead (read latency times requests over
// the kernel's time, counters of both batches), so a line's latency sets the copy rate, and copies
// issued in a burst stall the wave that issues them: one copy after every fourth to eighth MFMA of
// the multiplying wave (1,245 -> 1,189 us) beats the reading wave issuing them. Against one
// two-stage ring drained at every step (the kernel before it): 16384-token layer 1,466 -> 1,345
// us (1,315 with a reciprocal in place of silu's division), DeepSeek-V2-Lite-shaped 8192-token
// layer 1,307 -> 1,240, Qwen3-30B-A3B-shaped 4096-token layer 558 -> 502.
#include "lds_dma.h"
#include "pmpe_internal.h"

namespace pmpe {
namespace {

constexpr int BM = 256, BN = 256, BK = 64, THREADS = 512;
constexpr int HALF = 128 * 128;             // bytes of a half tile (128 rows x 64 bf16)
constexpr int STEP = 4 * HALF;              // one step's slots: A0 A1 B0 B1
constexpr int MAXG = 2 * PMPE_MAX_POOL + 1;  // routed experts + the shared group
constexpr int LIST = 256;                   // tiles of a block whose description is kept in LDS
constexpr int NRT = 4;                      // row_token slices in flight (see issue_rt)

template <int N>
constexpr std::integral_constant<int, N> ic{};

enum { G1 = 0, G1_SAVE = 1, G2 = 2, PLAIN = 3, GATHER = 4 };

struct TileInfo {
  int g;     // group: expert id, or E for the shared group
  int m0;    // first row of the tile within the group
  int n0;    // first output column
  int rows;  // valid rows (<= 256)
  int base;  // first row of the tile in the group's row space (permuted row / token)
};

// Two floats to a packed bf16 pair, round to nearest even (low half = a).
__device__ __forceinline__ uint32_t cvt_pk_bf16(float a, float b) {
  typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, b16x2));
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)uniform_ptr(p), 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}
constexpr uint32_t NO_STORE = 0x7FFFFFF0u;  // past every buffer's size: the store is dropped

template <int MODE>
__global__ __launch_bounds__(THREADS) void gemm256_kernel(FfnArgs a) {
  constexpr bool GATED = MODE == G1 || MODE == G1_SAVE, SAVE = MODE == G1_SAVE;
  constexpr bool AUDIT = MODE == G2, GATHER_A = MODE == GATHER;
  constexpr int NCOLS = GATED ? BN / 2 : BN;  // output columns per tile
  // Stores a wave issues for a tile with both A halves, by the phase of the last step that
  // they follow the copies of (S2..S4) and after that step (S5); for a tile without A1: S2, S5.
  constexpr int SQ = GATED ? (SAVE ? 5 : 1) : 1;  // per 16-row block and output half
  constexpr int S2 = GATED ? 0 : 4, S3 = GATED ? 2 * SQ : 4, S4 = GATED ? 2 * SQ : 4, S5 = 4 * SQ;
  constexpr int SALL = S2 + S3 + S4 + S5;
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * STEP];
  __shared__ __attribute__((aligned(16))) int s_rt[NRT][BM];
  __shared__ __attribute__((aligned(16))) int4 s_list[LIST];
  __shared__ int s_cum[MAXG + 1];
  __shared__ int s_cnt[MAXG];
  __shared__ int s_off[MAXG];
  __shared__ int s_perm[MAXG];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int E = a.n_pub + a.n_priv;
  const int ngroups = E + (a.Is > 0 ? 1 : 0);
  const int H = a.H;
  const int TK = a.T * a.k;

  if (tid < 64) {
    // Tile order: the shared group first (all T tokens; in GEMM2 its K loop over 2 I_s is the
    // longest, so its tiles must not be left for the end), then the public and the private
    // experts interleaved (mixed_position): each XCD's slice then holds full and half-filled
    // tiles alike, while the tiles of one expert stay adjacent.
    const int sh = (ngroups > E) ? 1 : 0;
    for (int g = tid; g < ngroups; g += 64) s_perm[g < E ? sh + mixed_position(g, a.n_pub, a.n_priv) : 0] = g;
    // (this wave's LDS writes above precede its reads below)
    int running = 0;
    for (int o0 = 0; o0 < ngroups; o0 += 64) {
      const int o = o0 + tid;
      int nt = 0;
      if (o < ngroups) {
        const int g = s_perm[o];
        const int cnt = (g < E) ? a.count[g] : a.T;
        s_cnt[g] = cnt;
        s_off[g] = (g < E) ? a.offset[g] : 0;
        const int width = GATED ? ((g < E) ? a.I : a.Is) : H;
        nt = ((cnt + BM - 1) / BM) * ((width + NCOLS - 1) / NCOLS);
      }
      const int incl = wave_incl_scan(nt);
      if (o < ngroups) s_cum[o + 1] = running + incl;
      running += __shfl(incl, 63, 64);
    }
    if (tid == 0) s_cum[0] = 0;
  }
  __syncthreads();

  // Block ids are remapped so that XCD x (workgroups go to the 8 XCDs round-robin) takes one
  // contiguous slice of the routed tiles, dealt round-robin to its blocks: tiles that share an
  // expert's weights or rows then run on one XCD and meet in its L2. The shared group's tiles
  // come before them in every XCD's list, dealt to the XCDs in chunks of XCH consecutive tiles
  // (M tiles of one weight tile), so that every XCD gets its share of them.
  constexpr int XCH = 8;
  const int total = s_cum[ngroups];
  const int n_sh = (ngroups > E) ? s_cum[1] : 0;  // shared tiles, first in the order
  const int n_rt = total - n_sh;
  const int b = blockIdx.x, x = b & 7, q = b >> 3;
  const int nbx = ((int)gridDim.x - x + 7) >> 3;
  const int nch = (n_sh + XCH - 1) / XCH;               // chunks of shared tiles
  const int nch_x = (nch > x) ? (nch - x + 7) / 8 : 0;  // those of XCD x
  // the last chunk (nch - 1) is the only one that may be partial
  const int sh_x = nch_x * XCH - ((nch_x > 0 && (nch - 1) % 8 == x) ? (nch * XCH - n_sh) : 0);
  const int cnt_x = sh_x + (n_rt >> 3) + (x < (n_rt & 7) ? 1 : 0);
  const int start_x = n_sh + x * (n_rt >> 3) + min(x, n_rt & 7);
  const int ntl = (cnt_x > q && q < nbx) ? (cnt_x - q + nbx - 1) / nbx : 0;
  if (ntl == 0) return;

  // tile i of this block: (g | rows << 16, m0, n0, base)
  auto find_tile = [&](int i) {
    const int j = q + i * nbx;  // index within the XCD's tiles
    const int L = (j < sh_x) ? (x + 8 * (j / XCH)) * XCH + (j % XCH) : start_x + (j - sh_x);
    int lo = 0, hi = ngroups - 1;  // last position o with s_cum[o] <= L (a group with tiles)
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_cum[mid] <= L) lo = mid; else hi = mid - 1;
    }
    const int g = s_perm[lo], cnt = s_cnt[g];
    const int mt = (cnt + BM - 1) / BM;
    const int local = L - s_cum[lo];
    const int ntn = (s_cum[lo + 1] - s_cum[lo]) / mt;  // N tiles
    // Routed experts: chunks of c M tiles against every N tile, so that the 32 tiles an XCD runs
    // at a time are about 5 x 6 and not 16 x 2 (operands fetched once per XCD: 12 against 18
    // per 32 tiles; 16384-token layer 1,227 -> 1,202 us). The shared group goes by XCH below.
    const int c = (g < E) ? max(4, 32 / ntn) : mt;
    const int ch = local / (c * ntn), rem = local - ch * (c * ntn);
    const int mc = min(c, mt - ch * c);
    const int n = rem / mc, m = ch * c + (rem - n * mc);
    return make_int4(g | (min(BM, cnt - m * BM) << 16), m * BM, n * NCOLS, s_off[g] + m * BM);
  };
  for (int i = tid; i < min(ntl, LIST); i += THREADS) s_list[i] = find_tile(i);
  __syncthreads();
  auto tile_of = [&](int i) {
    const int4 v = (i < LIST) ? s_list[i] : find_tile(i);
    const int gr = __builtin_amdgcn_readfirstlane(v.x);
    return TileInfo{gr & 0xFFFF, __builtin_amdgcn_readfirstlane(v.y), __builtin_amdgcn_readfirstlane(v.z), gr >> 16,
                    __builtin_amdgcn_readfirstlane(v.w)};
  };
  // Does tile t read row_token? (gathered x rows in GEMM1; the audit in GEMM2)
  auto needs_rt = [&](const TileInfo& t) {
    if (t.g >= E) return false;
    return GATED ? (a.x_perm == nullptr) : (GATHER_A || (AUDIT && t.g >= a.n_pub));
  };
  const uint32_t lds0 = lds_addr(smem);
  const uint32_t rt0 = lds_addr(&s_rt[0][0]);
  // Copy row_token[base .. base + 256) of tile t into s_rt[slot] (wave 0; clamped reads). A
  // tile's slice is copied one tile before the producer reaches it. The producer is two
  // steps ahead of the consumer, whose tile's slice the audit still reads: with one step per
  // tile the slices of tiles ci .. ci + 3 are live. A gathering tile has at least two steps
  // (K = H >= 128), so its slice is older than copies that were waited for before it is read.
  auto issue_rt = [&](const TileInfo& t, int slot) {
    if (wave == 0 && needs_rt(t)) {
#pragma unroll
      for (int j = 0; j < BM / 64; ++j) {
        const int idx = min(t.base + j * 64 + lane, TK - 1);
        dma4(a.row_token + idx, rt0 + (slot * BM + j * 64) * 4);
      }
    }
  };

  // Producer: source offsets (bytes) of this lane's copies for the tile whose steps are being
  // issued. A copy instruction fills 8 rows of a half tile; wave w fills rows 16w .. 16w + 15.
  // Chunk c (16 bytes) of LDS row r holds logical chunk c ^ (r & 7), so that fragment reads of
  // 8 consecutive rows at one logical chunk cover the banks once.
  const int crow = wave * 16 + (lane >> 3);  // LDS row of copy 0 (copy 1: + 8)
  const uint32_t cchunk = (uint32_t)(((lane & 7) ^ (lane >> 3)) * 16);
  // weight row held by LDS row r of a half: within 32 rows, row 16 nb + j holds 8 (j / 4) + 4 nb + j % 4
  auto bperm = [](int r) { return (r & ~31) + 8 * ((r >> 2) & 3) + 4 * ((r >> 4) & 1) + (r & 3); };
  uint32_t offA[4], offB[4];  // [half * 2 + copy]
  const unsigned char* baseA = nullptr;
  const unsigned char* baseB = nullptr;
  int p_full = 0;  // the producer's tile has more than 128 rows
  auto setup = [&](const TileInfo& t, int slot) {
    const bool shared = t.g >= E;
    const bool priv = !shared && t.g >= a.n_pub;
    const int I = shared ? a.Is : a.I;
    const int K = GATED ? H : I;
    const unsigned char* w;
    if (shared) {
      w = (const unsigned char*)(GATED ? a.w13_sh : a.w2_sh);
    } else if (!priv) {
      w = (const unsigned char*)(GATED ? a.w13_pub : a.w2_pub) + (size_t)t.g * (GATED ? 2 : 1) * I * H * 2;
    } else {
      w = (const unsigned char*)(GATED ? a.w13_priv : a.w2_priv);
      if (w) w += (size_t)(t.g - a.n_pub) * (GATED ? 2 : 1) * I * H * 2;
    }
    // private rows without private weights: the copies read public rows, nothing is computed
    if (w == nullptr || (priv && (a.w13_priv == nullptr || a.w2_priv == nullptr)))
      w = (const unsigned char*)(GATED ? a.w13_pub : a.w2_pub);
    baseB = w;
    if (GATED)
      baseA = (const unsigned char*)((!shared && a.x_perm) ? a.x_perm : a.x);
    else
      baseA = (const unsigned char*)(GATHER_A ? a.x : shared ? a.h_sh : a.h);
    p_full = t.rows > 128;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = (i >> 1) * 128 + crow + (i & 1) * 8;
      const int rr = min(r, t.rows - 1);  // rows past the valid count reload a valid row
      uint32_t row = (uint32_t)(t.base + rr);
      if (GATED ? (!shared && !a.x_perm) : GATHER_A) row = (uint32_t)s_rt[slot][rr];
      offA[i] = row * (uint32_t)(K * 2) + cchunk;
      const int c = bperm(crow + (i & 1) * 8);
      int wrow;
      if (GATED)
        wrow = (i >> 1) * I + min(t.n0 + c, I - 1);
      else
        wrow = min(t.n0 + (i >> 1) * 128 + c, H - 1);
      offB[i] = (uint32_t)wrow * (uint32_t)(K * 2) + cchunk;
    }
    return K / BK;
  };
  // Copies of half h of A or B of the producer's current step (pk) into buffer `buf`.
  int pi = 0, pk = 0, pnk = 0;
  auto copyA1 = [&](auto h, auto i, uint32_t buf) {
    const uint32_t dst = lds0 + buf + h.value * HALF + wave * 2048;
    dma16s<i.value * 1024, false>(offA[h.value * 2 + i.value], baseA + pk * (BK * 2), dst);
  };
  auto copyB1 = [&](auto h, auto i, uint32_t buf) {
    const uint32_t dst = lds0 + buf + (2 + h.value) * HALF + wave * 2048;
    dma16s<i.value * 1024, false>(offB[h.value * 2 + i.value], baseB + pk * (BK * 2), dst);
  };
  auto copyA = [&](auto h, uint32_t buf) { copyA1(h, ic<0>, buf); copyA1(h, ic<1>, buf); };
  auto copyB = [&](auto h, uint32_t buf) { copyB1(h, ic<0>, buf); copyB1(h, ic<1>, buf); };
  constexpr std::integral_constant<int, 0> h0{};
  constexpr std::integral_constant<int, 1> h1{};
  // Move to the next step to issue; its kind: 0 none left, 1 without A1, 2 with A1.
  auto next_step = [&]() {
    if (pi >= ntl) return 0;
    if (pk == pnk) {  // the next tile; its gather indices arrived earlier
      ++pi;
      pk = 0;
      if (pi >= ntl) return 0;
      pnk = setup(tile_of(pi), pi % NRT);
      if (pi + 1 < ntl) issue_rt(tile_of(pi + 1), (pi + 1) % NRT);
    }
    return 1 + p_full;
  };
  // prologue: gather indices of tiles 0 and 1, then steps 0 and 1
  issue_rt(tile_of(0), 0);
  if (ntl > 1) issue_rt(tile_of(1), 1);
  wait_vmcnt<0>();
  __syncthreads();
  pnk = setup(tile_of(0), 0);
  int kind1 = 0, kind2 = 0;  // kinds of the steps one and two after the consumer's
  // A step's A1 is copied one consumer step after its other half tiles (in the first phase), so
  // that a phase issues one half tile; `late` is set while it is outstanding.
  bool late = false;
  auto copy_late = [&](uint32_t buf) {
    if (late) copyA(h1, buf);
    late = false;
  };
  auto copy_step = [&](uint32_t buf) {
    const int kind = next_step();
    if (kind) {
      copyA(h0, buf);
      copyB(h0, buf);
      copyB(h1, buf);
    }
    return kind;
  };
  late = copy_step(0) == 2;
  copy_late(0);
  ++pk;
  kind1 = copy_step(STEP);
  late = kind1 == 2;
  wait_vmcnt<0>();
  barrier_raw();
  if (wm == 1) barrier_raw();  // the second row group runs half a phase behind

  // Fragment addresses: row (lane & 15) of a 16-row block, K chunk 4 sub + lane / 16.
  const uint32_t lane_off = (uint32_t)((lane & 15) * 128 + (((lane >> 4) ^ (lane & 7)) << 4));
  uint32_t cbuf = 0;  // the consumer's buffer (0 or STEP)
  bf16x8 fa[4][2], fb0[2][2], fb1[2][2];
  // Wave wm's 16-row blocks of an A half are blocks 2 mb + wm, so a partly filled half loads
  // both row groups alike.
  auto readA = [&](auto h) {
    const uint32_t p0 = lane_off + cbuf + wm * 2048, p1 = p0 ^ 64;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      fa[mb][0] = as_bf16x8(*(const u32x4*)(smem + p0 + h.value * HALF + mb * 4096));
      fa[mb][1] = as_bf16x8(*(const u32x4*)(smem + p1 + h.value * HALF + mb * 4096));
    }
  };
  auto readB = [&](auto h, bf16x8 (&fb)[2][2]) {
    const uint32_t p0 = lane_off + cbuf + wn * 4096, p1 = p0 ^ 64;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      fb[nb][0] = as_bf16x8(*(const u32x4*)(smem + p0 + (2 + h.value) * HALF + nb * 2048));
      fb[nb][1] = as_bf16x8(*(const u32x4*)(smem + p1 + (2 + h.value) * HALF + nb * 2048));
    }
  };
  // Output stores share the counter of the copies. They follow the copies of the last step of
  // a tile, so for the next steps they are younger than the copies waited for and may stay in
  // flight: `fresh` is 2 and 1 in the two steps after a tile that stored (fst: its A halves).
  // Every wave issues the same number of stores whatever the valid rows (see epilogue).
  int fresh = 0, fst = 0;
  // Wait until at most N copies (and B2 or B1 stores, when `past`) are in flight.
  auto wait_copies = [&](auto n, auto b2, auto b1, bool past) {
    constexpr int N = decltype(n)::value, B2 = decltype(b2)::value, B1 = decltype(b1)::value;
    if (!past)
      wait_vmcnt<N>();
    else if (fst == 2)
      wait_vmcnt<N + B2>();
    else
      wait_vmcnt<N + B1>();
  };
  // End of a step: the half tiles that the next step's first phase reads have landed (A0 and
  // B0; without A1 also B1). Younger: the next step's B1 and A1, and the step after it. In a
  // tile's last step `stored` counts the stores it has issued.
  auto wait_next = [&](auto stored, bool last, auto n2) {
    constexpr int N2 = decltype(n2)::value;
    constexpr int SL = decltype(stored)::value;
    if (kind1 == 0 || kind2 == 0) {
      wait_vmcnt<0>();
    } else if (kind1 == 2) {
      if (last)
        wait_vmcnt<N2 + SL>();
      else
        wait_copies(ic<N2>, ic<S4 + S5>, ic<S5>, fresh == 2);
    } else {
      if (last)
        wait_vmcnt<N2 - 4 + SL>();
      else
        wait_copies(ic<N2 - 4>, ic<S5>, ic<S5>, fresh == 2);
    }
  };
  // reads of this phase are done, and the waits above hold for every wave of the block
  auto phase_mid = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    barrier_raw();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
  };
  auto phase_end = [&]() {
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    barrier_raw();
    __builtin_amdgcn_sched_barrier(0);
  };
  // the first MB row blocks of a quadrant
  auto mul = [&](auto blocks, f32x4 (&acc)[4][2], const bf16x8 (&fb)[2][2]) {
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int mb = 0; mb < decltype(blocks)::value; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[nb][sub], fa[mb][sub], acc[mb][nb], 0, 0, 0);
  };
  // the same with copies issued between the MFMAs
  auto mulc_mb = [&](auto blocks, f32x4 (&acc)[4][2], const bf16x8 (&fb)[2][2], auto&& copy) {
    constexpr int MB = decltype(blocks)::value;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[nb][sub], fa[mb][sub], acc[mb][nb], 0, 0, 0);
        if (sub == 0 && mb == (MB - 1) / 2) {
          __builtin_amdgcn_sched_barrier(0);
          copy(ic<0>);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (sub == 1 && mb == (MB - 1) / 2) {
          __builtin_amdgcn_sched_barrier(0);
          copy(ic<1>);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  auto mulc = [&](f32x4 (&acc)[4][2], const bf16x8 (&fb)[2][2], auto&& copy) { mulc_mb(ic<4>, acc, fb, copy); };
  auto end_step = [&]() {
    cbuf ^= STEP;
    kind1 = kind2;
    fresh = max(fresh - 1, 0);
  };

  // K loop and output of one tile; halves: A halves with valid rows (0: nothing is computed);
  // blocks: row blocks per wave of the last of them that may hold valid rows.
  auto tile_body = [&](auto halves, auto blocks, const TileInfo& ct, int cnk, void* out, int ld, int width) {
    constexpr int AH = decltype(halves)::value, BLOCKS = decltype(blocks)::value;
    f32x4 acc[AH > 0 ? AH : 1][2][4][2];  // [A half][B half][row block][column block]
#pragma unroll
    for (int i = 0; i < AH; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
          for (int nb = 0; nb < 2; ++nb) acc[i][j][mb][nb] = f32x4{0, 0, 0, 0};
    // Output of row blocks MB0 .. MB1 - 1 of A half i (and, not GATED, of column half j). A lane
    // holds columns 8 (lane / 16) .. + 7 (blocks nb = 0, 1) of row lane % 16 of a block. Rows
    // past the valid count lie past the buffer's size, columns past the width are sent there:
    // the hardware drops both, so the number of stores is fixed. A quadrant is stored in the
    // reading half of a later phase, while the other row group multiplies; storing the whole
    // tile after its last step instead held both row groups up in turn.
    const bool save = SAVE && ct.g < E;
    auto store = [&](auto ih, auto jh, auto mb0, auto mb1) {
      constexpr int i = decltype(ih)::value, j = decltype(jh)::value;
      // opaque copies, so that the addresses are formed here and not kept in registers
      // through the K loop
      int ln = lane, row0 = ct.base;
      asm volatile("" : "+v"(ln));
      asm volatile("" : "+s"(row0));
      const __amdgpu_buffer_rsrc_t ro = buffer((const uint16_t*)out + (size_t)row0 * ld, (uint32_t)(ct.rows * ld * 2));
      const int c = ct.n0 + j * 128 + wn * 32 + (ln >> 4) * 8;
#pragma unroll
      for (int mb = decltype(mb0)::value; mb < decltype(mb1)::value; ++mb) {
        const int r = i * 128 + (2 * mb + wm) * 16 + (ln & 15);
        u32x4 o;
        if constexpr (GATED) {
          const f32x4 g0 = acc[i][0][mb][0], g1 = acc[i][0][mb][1], u0 = acc[i][1][mb][0], u1 = acc[i][1][mb][1];
          const float g[8] = {g0[0], g0[1], g0[2], g0[3], g1[0], g1[1], g1[2], g1[3]};
          float v[8];
          silu_n<8>(g, v);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[e] *= u0[e];
            v[4 + e] *= u1[e];
          }
          o = u32x4{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]), cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7])};
          if (save) {
            const __amdgpu_buffer_rsrc_t rs = buffer(a.ab_save + (size_t)row0 * (2 * width), (uint32_t)(ct.rows * 2 * width * 4));
            const uint32_t p = c < width ? (uint32_t)((r * 2 * width + c) * 4) : NO_STORE, pu = c < width ? p + (uint32_t)width * 4 : NO_STORE;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, g0), rs, p, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, g1), rs, p + (c < width ? 16 : 0), 0, 0);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, u0), rs, pu, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, u1), rs, pu + (c < width ? 16 : 0), 0, 0);
          }
        } else {
          const f32x4 v0 = acc[i][j][mb][0], v1 = acc[i][j][mb][1];
          o = u32x4{cvt_pk_bf16(v0[0], v0[1]), cvt_pk_bf16(v0[2], v0[3]), cvt_pk_bf16(v1[0], v1[1]), cvt_pk_bf16(v1[2], v1[3])};
        }
        __builtin_amdgcn_raw_buffer_store_b128(o, ro, c < width ? (uint32_t)((r * ld + c) * 2) : NO_STORE, 0, 0);
      }
    };
    for (int kc = 0; kc < cnk; ++kc) {
      const bool last = kc == cnk - 1;
      if constexpr (AH == 2) {
        readA(h0);
        readB(h0, fb0);
        // B1 of this step landed; younger: its A1 and the next step
        if (kind1)
          wait_copies(ic<8>, ic<S5>, ic<S5>, fresh > 0);
        else
          wait_vmcnt<2>();
        phase_mid();
        mulc(acc[0][0], fb0, [&](auto i) { if (late) copyA1(h1, i, cbuf ^ STEP); });
        if (kind1) ++pk;
        phase_end();

        kind2 = next_step();
        readB(h1, fb1);
        if constexpr (!GATED)
          if (last) store(h0, h0, ic<0>, ic<4>);
        // A1 of this step landed; younger: the next step
        if (kind1 == 2)
          wait_copies(ic<8>, ic<SALL>, ic<S5>, fresh == 2);
        else if (kind1 == 1)
          wait_vmcnt<6>();
        else
          wait_vmcnt<0>();
        phase_mid();
        mulc(acc[0][1], fb1, [&](auto i) { if (kind2) copyA1(h0, i, cbuf); });
        phase_end();

        late = kind2 == 2;
        readA(h1);
        if (last) {
          if constexpr (GATED)
            store(h0, h0, ic<0>, ic<2>);
          else
            store(h0, h1, ic<0>, ic<4>);
        }
        if constexpr (BLOCKS <= 2) {
          // few row blocks in the second half: its two quadrants in one phase
          wait_next(ic<S2 + (SAVE ? 2 : S3)>, last, ic<6>);
          phase_mid();
          mulc_mb(blocks, acc[1][1], fb1, [&](auto i) { if (kind2) copyB1(h0, i, cbuf); });
          mulc_mb(blocks, acc[1][0], fb0, [&](auto i) { if (kind2) copyB1(h1, i, cbuf); });
          phase_end();
          if (last) {
            if constexpr (GATED)
              store(h0, h0, ic<2>, ic<4>);
            else
              store(h1, h1, ic<0>, ic<4>);
          }
        } else {
          phase_mid();
          mulc_mb(blocks, acc[1][1], fb1, [&](auto i) { if (kind2) copyB1(h0, i, cbuf); });
          phase_end();

          if (last) {
            if constexpr (GATED)
              store(h0, h0, ic<2>, ic<4>);
            else
              store(h1, h1, ic<0>, ic<4>);
          }
          wait_next(ic<S2 + (SAVE ? 4 : S3 + S4)>, last, ic<8>);
          phase_mid();
          mulc_mb(blocks, acc[1][0], fb0, [&](auto i) { if (kind2) copyB1(h1, i, cbuf); });
          phase_end();
        }
        if (last) store(h1, h0, ic<0>, ic<4>);
      } else {
        copy_late(cbuf ^ STEP);
        if (kind1) ++pk;
        if constexpr (AH == 1) {
          readA(h0);
          readB(h0, fb0);
          readB(h1, fb1);
        }
        phase_mid();
        if constexpr (AH == 1) mul(blocks, acc[0][0], fb0);
        phase_end();
        kind2 = next_step();
        if (kind2) {
          copyA(h0, cbuf);
          copyB(h0, cbuf);
        }
        late = kind2 == 2;
        if constexpr (AH == 1 && !GATED)
          if (last) store(h0, h0, ic<0>, ic<4>);
        wait_next(ic<AH == 1 ? S2 : 0>, last, ic<8>);
        phase_mid();
        if constexpr (AH == 1) mulc_mb(blocks, acc[0][1], fb1, [&](auto i) { if (kind2) copyB1(h1, i, cbuf); });
        else if (kind2) copyB(h1, cbuf);
        phase_end();
        if constexpr (AH == 1)
          if (last) store(h0, ic<GATED ? 0 : 1>, ic<0>, ic<4>);
      }
      end_step();
    }
    fst = AH;
    // (a shared tile of the saving variant stores no projections: no allowance)
    fresh = (AH > 0 && (!SAVE || save)) ? 2 : 0;
    __builtin_amdgcn_sched_barrier(0);
  };

  for (int ci = 0; ci < ntl; ++ci) {
    const TileInfo ct = tile_of(ci);
    const bool c_shared = ct.g >= E;
    const bool c_priv = !c_shared && ct.g >= a.n_pub;
    const int cI = c_shared ? a.Is : a.I;
    const int cnk = (GATED ? H : cI) / BK;
    const bool c_valid = !(c_priv && (a.w13_priv == nullptr || a.w2_priv == nullptr));
    const int width = GATED ? cI : H;
    void* out = GATED ? (c_shared ? a.h_sh : a.h) : (c_shared ? a.y_shared : a.y_perm);
    if (!c_valid)
      tile_body(ic<0>, ic<0>, ct, cnk, out, width, width);
    else if (ct.rows <= 64)
      tile_body(ic<1>, ic<2>, ct, cnk, out, width, width);
    else if (ct.rows <= 128)
      tile_body(ic<1>, ic<4>, ct, cnk, out, width, width);
    else if (ct.rows <= 160)
      tile_body(ic<2>, ic<1>, ct, cnk, out, width, width);
    else if (ct.rows <= 192)
      tile_body(ic<2>, ic<2>, ct, cnk, out, width, width);
    else
      tile_body(ic<2>, ic<4>, ct, cnk, out, width, width);
    if (!c_valid && !GATED) {
      // private rows without private weights: not executed, not audited, y zeroed
      if (tid == 0 && a.dev_status) atomicOr(a.dev_status, PMPE_DEV_PRIV_WEIGHTS_MISSING);
      constexpr int VPR = NCOLS / 8;
      for (int i = tid; i < ct.rows * VPR; i += THREADS) {
        const int r = i / VPR, c = ct.n0 + (i - r * VPR) * 8;
        if (c < width) *(u32x4*)((uint16_t*)out + (size_t)(ct.base + r) * width + c) = u32x4{0, 0, 0, 0};
      }
    }
    // Execution audit: the first N tile of every executed private M tile counts its rows.
    if (AUDIT && c_priv && c_valid && ct.n0 == 0) {
      if (tid < ct.rows) atomicAdd(&a.audit_rows[s_rt[ci % NRT][tid]], 1u);
      if (ct.m0 == 0 && tid == 0 && a.audit_calls) atomicAdd(&a.audit_calls[ct.g - a.n_pub], 1u);
    }
  }
  wait_vmcnt<0>();             // no copy may still be writing LDS when the block exits
  if (wm == 0) barrier_raw();  // both row groups pass the same number of barriers
}

int cu_count() {
  int dev = 0, v = 0;
  if (hipGetDevice(&dev) == hipSuccess &&
      hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
    return v;
  return 256;
}

template <int MODE>
hipError_t launch(const FfnArgs& a, hipStream_t s) {
  // Persistent grid: one block per CU (a multiple of the 8 XCDs), never more than the tiles
  // there can be.
  constexpr bool GATED = MODE == G1 || MODE == G1_SAVE;
  constexpr int NCOLS = GATED ? BN / 2 : BN;
  const int E = a.n_pub + a.n_priv;
  const int64_t w = GATED ? a.I : a.H;
  int64_t tiles = ((int64_t)a.T * a.k / BM + E) * ((w + NCOLS - 1) / NCOLS);
  if (a.Is > 0) {
    const int64_t ws = GATED ? a.Is : a.H;
    tiles += ((a.T + BM - 1) / BM) * ((ws + NCOLS - 1) / NCOLS);
  }
  int64_t g = cu_count();
  if (tiles < g) g = (tiles + 7) / 8 * 8;
  hipLaunchKernelGGL(gemm256_kernel<MODE>, dim3((unsigned)g), dim3(THREADS), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm256_up(const FfnArgs& a, hipStream_t s) {
  return a.ab_save ? launch<G1_SAVE>(a, s) : launch<G1>(a, s);
}
hipError_t launch_gemm256_down(const FfnArgs& a, hipStream_t s) { return launch<G2>(a, s); }
hipError_t launch_gemm256_plain(const FfnArgs& a, hipStream_t s) {
  return a.gather_a ? launch<GATHER>(a, s) : launch<PLAIN>(a, s);
}

}  // namespace pmpe
