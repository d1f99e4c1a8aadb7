// Grouped expert GEMMs of the sparsified MoE output (Eq. ace_sparse_output):
// every kept slot (token t, expert e) evaluates the SwiGLU expert of
// Eq. swiglu_expert, f_e(x) = W_down (SiLU(W_gate x) * (W_up x)), in nn.Linear
// layouts.  Rows are the compacted kept slots of the dispatch plan, grouped by
// expert, so every M tile multiplies rows of one expert against that expert's
// weights.
//
//   gateup: H[r, :] = SiLU(x_in[perm[r]] W_gate[e]^T) * (x_in[perm[r]] W_up[e]^T)
//           (A rows gathered through perm; SiLU and the product fused into the
//           epilogue)
//   down:   Y[r, :] = H[r, :] W_down[e]^T
//
// bf16 path (MI355X, bf16 MFMA v_mfma_f32_16x16x32_bf16, fp32 accumulation).
// With 50% of 32768 slots kept over 128 experts an expert sees ~90-190 rows, so
// the layer streams every activated expert's weights once and is HBM-bound:
//  * an M tile holds up to 256 rows, so an expert's weights are read once per
//    tile (a 128-row tile would re-read them for every expert past 128 rows);
//    the row count selects one of four unrolled bodies (64..256 rows) so MFMAs
//    and loads are issued only for the 16-row blocks a tile has;
//  * operands move HBM/L2 -> LDS with global_load_lds_dwordx4 (no VGPR staging)
//    through two LDS rings in 160 KB: activations (L2-resident) 2-4 K stages deep,
//    expert weights (from HBM; with the non-temporal hint when no other M tile
//    reads them) 3-8 stages deep; each wave waits only for the
//    stage it computes next (vmcnt counted exactly from the issue schedule, in closed
//    form: one of two constants with two activation stages, else of a few, since a
//    64-way choice is a branch tree that costs matrix-bound tiles several percent),
//    then one barrier per K step;
//  * one DMA instruction moves 8 rows x 128 bytes (whole cache lines) and lane i
//    lands at byte 16*i; the chunk a lane fetches is XOR-swizzled by its row so
//    the MFMA fragment reads (16 rows x 16 bytes) are bank-conflict free;
//  * 8 waves (two per SIMD, so one wave's LDS reads overlap the other's MFMAs)
//    as 4 x 2: a wave owns a quarter of the row blocks (interleaved, so short
//    tiles stay balanced) and two column groups (gate/up: gate and up blocks of
//    the same 16 features, so SwiGLU happens in registers; down: 32 columns);
//  * the down launch gives each workgroup two N tiles of one M tile, run as one
//    pipeline (the second tile's first stages load under the first's last steps).
// fp32 path: the same tile body on 32-wide K stages, four v_mfma_f32_16x16x4f32 per
// pair of fragments.  By the peak rates an fp32 multiply takes 16 times the matrix time
// of a bf16 one, 8 times per byte of operand, so the matrix cores bound all but the
// shortest tiles, and what counts is to spread the work evenly: M tiles of 64 rows (the
// plan's tile size for fp32 layers), 32 features or 64 columns wide, half the LDS each, so
// two workgroups share a CU and one's ramp and stores run under the other's K loop.  The kernels that loaded one
// 16-wide K step at a time between barriers took 199 + 105 us for 517 tokens (1024
// hidden, 32 experts of 512, top-4), 256-row tiles with all of the LDS 63 + 35, half
// of it 53 + 29; 929 tokens on 11 experts take 159 us a layer with 256-row tiles,
// 120 with 64-row ones.  Tiles twice as wide leave CUs idle (929 tokens: 270 us).
//
// Launch order is XCD-aware: workgroups are dealt to the 8 XCDs round-robin, so
// block b runs on XCD b % 8; the N tiles of one M tile are mapped to one XCD so
// the activation rows they share stay in that XCD's L2.
#include "gemm_pipe.h"
#include "lds_dma.h"

namespace ace {

namespace {

constexpr int kFragBytes = kUnitBytes;  // one staged unit (8 rows x 64 bf16, or 16 rows x 32)
static_assert(kFragBytes == kPipeUnitBytes, "one DMA unit per fragment");

struct TileInfo {
  int e, row0, rows;
  bool valid;
  bool sh;    // a tile of the appended dense expert
  bool once;  // no other M tile of this launch reads this tile's expert weights
};

__device__ __forceinline__ void map_block(int b, int nN, int *grp, int *nt) {
  const int xcd = b & 7;
  const int j = b >> 3;
  *grp = xcd + 8 * (j / nN);
  *nt = j % nN;
}

// TM: rows of an M tile
template <int TM> __device__ __forceinline__ TileInfo tile_info(const GemmArgs &a, int grp) {
  TileInfo ti;
  ti.sh = false;
  if (a.dense_rows > 0) {
    ti.e = 0;
    ti.row0 = grp * TM;
    ti.rows = min(TM, a.dense_rows - ti.row0);
    ti.valid = ti.rows > 0;
    ti.once = a.dense_rows <= TM;
  } else {
    const int nr = a.n_tiles[0];
    if (a.tile_order && grp < nr) grp = a.tile_order[grp];
    ti.valid = grp < nr;
    ti.e = ti.valid ? a.tile_expert[grp] : 0;
    ti.row0 = ti.valid ? a.tile_row0[grp] : 0;
    ti.rows = ti.valid ? a.tile_rows[grp] : 0;
    // an expert's tiles are consecutive in the list
    ti.once = ti.valid && !(grp > 0 && a.tile_expert[grp - 1] == ti.e) &&
              !(grp + 1 < nr && a.tile_expert[grp + 1] == ti.e);
    if (!ti.valid && grp - nr < a.sh_tiles) {
      ti.sh = true;
      ti.e = 0;
      ti.row0 = (grp - nr) * TM;
      ti.rows = min(TM, a.sh_rows - ti.row0);
      ti.valid = ti.rows > 0;
      ti.once = a.sh_tiles == 1;
    }
  }
  return ti;
}

constexpr int kGemmWaves = 8;  // waves per workgroup (two per SIMD)
// 32-wide k halves per pipeline stage.  Two (64-wide stages) measured faster than
// one with deeper rings: the stream rate, not the bytes in flight, is the limit.
template <int CG> constexpr int stage_halves() { return 2; }

// Pipe, Closed and Pending (gemm_pipe.h): ring depths per tile shape and the exact
// wait counts of a wave's DMA issue sequence.

// Output stores of gemm_tile: lane holds column r16 of each block, rows 4*g + q.
template <typename T, bool GATEUP, int MW, int CW, int RW, int BN>
__device__ __forceinline__ void store_tile_impl(int ld, const TileInfo &ti, void *outp,
                                                f32x4_t (&acc)[MW][2 * CW], int nt, int wr, int wc, int r16, int g) {
#pragma unroll
  for (int fl = 0; fl < CW; ++fl) {
    const int grp = wc * CW + fl;
    if (GATEUP) {
      T *H = static_cast<T *>(outp);
      const int f = nt * BN + grp * 16 + r16;
#pragma unroll
      for (int i = 0; i < MW; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = (wr + RW * i) * 16 + 4 * g + q;
          if (row < ti.rows)
            H[static_cast<size_t>(ti.row0 + row) * ld + f] = swiglu(acc[i][fl * 2][q], acc[i][fl * 2 + 1][q], T{});
        }
    } else {
      T *Y = static_cast<T *>(outp);
      const int n = nt * BN + grp * 32 + r16;
#pragma unroll
      for (int i = 0; i < MW; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = (wr + RW * i) * 16 + 4 * g + q;
          if (row < ti.rows) {
            T *yr = Y + static_cast<size_t>(ti.row0 + row) * ld + n;
            yr[0] = Elem<T>::from_f32(acc[i][fl * 2][q]);
            yr[16] = Elem<T>::from_f32(acc[i][fl * 2 + 1][q]);
          }
        }
    }
  }
}

// One M tile x ntiles (1 or 2) consecutive N tiles from nt0, with MB 16-row
// blocks, CG column groups and KH = 2 k halves per stage (64-wide stages: 128
// bytes of every row).  One DMA
// instruction moves an 8-row unit: 8 rows x 128 bytes, each row a whole cache
// line (16-row x 64-byte fragments touch twice as many lines per instruction and
// stream measurably slower).  A stage of A holds units u = 2 rb + j (row block
// rb, row half j), wave w staging u = w, w+W, ...; a stage of B holds units
// b = 2 (2 fg + cb) + j (column group fg, block cb (gate/up: 0 gate, 1 up;
// down: the group's two 16-column halves), row half j), wave w staging
// b = w*NB .. w*NB+NB-1.  Inside a unit, row r's 16-byte chunk c sits in slot
// c ^ r (both units of a block alike), so the MFMA fragment reads (16 rows, one
// chunk each) run at the full LDS rate.  Wave w computes row blocks wr, wr+RW,
// ... (wr = w/2) against the CG/2 column groups starting at wc*CG/2 (wc = w%2).
template <typename T, bool GATEUP, int MB, int CG, int KH, int W, bool OWN>
__device__ __forceinline__ void gemm_tile(const GemmArgs &a, const TileInfo &ti, int nt0, int ntiles, int erot,
                                          uint8_t *smem) {
  static_assert(KH == 2, "8-row DMA units span a 64-wide K stage");
  using P = Pipe<MB, CG, KH, W>;
  constexpr int RW = W / 2;    // waves along the rows
  constexpr int NAM = P::NA_MAX, NB = P::NB, SA = P::SA, SB = P::SB, BK = kStageElems<T>;
  typedef typename Frag<T>::type frag_t;
  constexpr int MW = MB / RW;  // row blocks per wave
  constexpr int CW = CG / 2;   // column groups per wave
  constexpr int BN = GATEUP ? 16 * CG : 32 * CG;  // tile width (features or output columns)
  static_assert(W % 2 == 0, "waves form an RW x 2 grid");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int wr = wave >> 1, wc = wave & 1;
  const int m = OWN && ti.sh ? a.sh_m : a.m;
  const int K = GATEUP ? a.d : m;
  // routed tile: the routed experts' operands; appended dense-expert tile: its own
  const T *act = static_cast<const T *>(ti.sh ? a.sh_act : a.act);
  const int32_t *perm = ti.sh ? nullptr : a.perm;
  const void *w0 = ti.sh ? a.sh_w0 : a.w0;
  const void *w1 = ti.sh ? a.sh_w1 : a.w1;
  void *outp = ti.sh ? a.sh_out : a.out;
  // A units this wave stages per stage (wave-uniform): only units holding a row of
  // the tile (unit u covers rows 8u .. 8u+7); the MFMAs below skip row blocks past
  // the tile too, and rows past the tile are never stored
  const int fav = min(P::FA, (ti.rows + 7) >> 3);
  const int na = fav > wave ? (fav - wave + W - 1) / W : 0;
  const int ur = lane >> 3;  // DMA lane -> row in its unit

  // A units this wave stages: u = wave + W j -> row block u / 2, row half u % 2 (=
  // wave % 2).  Their token rows come through perm (routed tiles).  The perm loads
  // are issued from inline assembly ahead of the weight prologue and waited for
  // explicitly after it: a compiler-placed wait for them would be a vmcnt(0),
  // which also waits for the weight DMAs issued in between and so holds the
  // activation prologue back by a whole memory round trip.
  int srow[NAM];
#pragma unroll
  for (int j = 0; j < NAM; ++j) {
    const int u = min(wave + W * j, P::FA - 1);
    const int row = min((u >> 1) * 16 + (u & 1) * 8 + ur, ti.rows - 1);  // rows past the tile repeat its last row
    srow[j] = perm ? gload_i32(perm + ti.row0 + row) : ti.row0 + row;
  }
  // B units this wave stages: b = wave * NB + t -> block b / 2, row half t % 2
  const T *bsrc[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const int b = wave * NB + t;
    const int blk = b >> 1, j = b & 1;
    const int fg = blk >> 1, cb = blk & 1;
    const int c = kChunkElems<T> * unit_chunk(lane);
    if (GATEUP) {
      const size_t f = static_cast<size_t>(ti.e) * m + nt0 * BN + fg * 16 + 8 * j + ur;
      bsrc[t] = static_cast<const T *>(cb ? w1 : w0) + f * a.d + c;
    } else {
      const size_t n = static_cast<size_t>(ti.e) * a.d + nt0 * BN + fg * 32 + cb * 16 + 8 * j + ur;
      bsrc[t] = static_cast<const T *>(w0) + n * K + c;
    }
  }
  // fragment read offsets inside a 16-row block (two units) for k halves 0 and 1
  const int rd_off0 = unit_read_offset(lane, 0), rd_off1 = unit_read_offset(lane, 1);
  const uint32_t ldsA = lds_addr(smem);
  const uint32_t ldsB = ldsA + SA * P::ASZ;
  const uint8_t *smemA = smem;
  const uint8_t *smemB = smem + SA * P::ASZ;

  f32x4_t acc[MW][2 * CW];
#pragma unroll
  for (int i = 0; i < MW; ++i)
#pragma unroll
    for (int c = 0; c < 2 * CW; ++c) acc[i][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto store_tile = [&](f32x4_t (&ac)[MW][2 * CW], int nt) {
    store_tile_impl<T, GATEUP, MW, CW, RW, BN>(GATEUP ? m : a.d, ti, outp, ac, nt, wr, wc, r16, g);
  };

  const int nk = K / BK;
  // ntiles (1 or 2) N tiles of the M tile, nt0 and nt0 + 1, run as one pipeline
  // of NK = ntiles * nk stages: stage s is K block s % nk of tile s / nk, so the
  // second tile's first stages are in flight while the first tile's last steps
  // and its output stores run (no second prologue ramp)
  const int NK = ntiles * nk;
  const size_t tile_step = static_cast<size_t>(BN) * K;  // weight elements from one N tile to the next
  // Pipeline stage s covers K block (s + k0) % nk, k0 set by the tile's expert.
  // Experts start at different K blocks: rows 4 KB apart (d = 2048 bf16) read at
  // one K offset by every workgroup at once concentrate on a few HBM channels and
  // stream ~20% slower.  Every tile of one expert keeps one K order: the N tiles
  // of an M tile share its activation rows in their XCD's L2, and the M tiles of a
  // large expert that run at the same time on one XCD share its weight rows
  // (starting each M tile at its own block left them out of step, and the
  // wider-pool gate/up fetched three times its weight bytes from beyond L2).
  const int k0 = erot % nk;
  auto kofs = [&](int s) {
    s = s < nk ? s : s - nk;
    return (s + k0 < nk ? s + k0 : s + k0 - nk) * BK;
  };
  // weight units of stage s into LDS stage base st: weights that no other M tile
  // reads stream with the non-temporal hint; weights shared by several M tiles
  // (large experts, the dense expert's tiles) stay cacheable for the other tiles
  auto issue_b = [&](uint32_t st, int s) {
    const size_t o = (s < nk ? 0 : tile_step) + kofs(s);
    if (ti.once) {
#pragma unroll
      for (int t = 0; t < NB; ++t) dma16_stream(bsrc[t] + o, st + (wave * NB + t) * kFragBytes);
    } else {
#pragma unroll
      for (int t = 0; t < NB; ++t) dma16(bsrc[t] + o, st + (wave * NB + t) * kFragBytes);
    }
  };
  // prologue: B stages 0..SB-2, then A stages 0..SA-2
  for (int s = 0; s < SB - 1 && s < NK; ++s) {
    const uint32_t st = ldsB + s * P::BSZ;
    issue_b(st, s);
  }
  if (perm) {
    // the perm loads, issued before these weight DMAs (a constant count unless K is
    // shorter than the weight prologue)
    if (NK >= SB - 1)
      wait_vmcnt((SB - 1) * NB);
    else
      wait_vmcnt(NK * NB);
#pragma unroll
    for (int j = 0; j < NAM; ++j) reg_ready(srow[j]);
  }
  const T *asrc[NAM];
#pragma unroll
  for (int j = 0; j < NAM; ++j) asrc[j] = act + static_cast<size_t>(srow[j]) * K + kChunkElems<T> * unit_chunk(lane);
  for (int s = 0; s < SA - 1 && s < NK; ++s) {
    const uint32_t st = ldsA + s * P::ASZ;
#pragma unroll
    for (int j = 0; j < NAM; ++j)
      if (j < na) dma16(asrc[j] + kofs(s), st + (wave + W * j) * kFragBytes);
  }

  using CF = Closed<P>;
  for (int kt = 0; kt < NK; ++kt) {
    if constexpr (CF::on) {  // bodies for more than 64 rows: every wave stages A units
      if (CF::nb_pending(kt, NK))
        wait_vmcnt(NB);
      else
        wait_vmcnt(0);
    } else {
      wait_vmcnt_in<0, Pending<P>::MAX>(Pending<P>::count(kt, NK, na));
    }
    barrier();  // stage kt landed for every wave; every wave is done with stage kt-1
    if (kt + SA - 1 < NK) {
      const int s = kt + SA - 1;
      const uint32_t st = ldsA + (s % SA) * P::ASZ;
#pragma unroll
      for (int j = 0; j < NAM; ++j)
        if (j < na) dma16(asrc[j] + kofs(s), st + (wave + W * j) * kFragBytes);
    }
    const uint8_t *sa = smemA + (kt % SA) * P::ASZ;
    const uint8_t *sb = smemB + (kt % SB) * P::BSZ;
#pragma unroll
    for (int h = 0; h < KH; ++h) {
      frag_t bf[2 * CW];  // [fl * 2 + cb]: column group wc*CW + fl, block cb
#pragma unroll
      for (int c = 0; c < 2 * CW; ++c)
        bf[c] = *reinterpret_cast<const frag_t *>(sb + (2 * (wc * CW + (c >> 1)) + (c & 1)) * 2 * kFragBytes +
                                                    (h ? rd_off1 : rd_off0));
      // every row block's fragment is read up front, with the weight fragments
      // (blocks past the tile read stale LDS and are not multiplied): a read
      // placed after the branch below made each row block's MFMAs wait a full
      // LDS round trip
      frag_t av[MW];
#pragma unroll
      for (int i = 0; i < MW; ++i)
        av[i] = *reinterpret_cast<const frag_t *>(sa + (wr + RW * i) * 2 * kFragBytes + (h ? rd_off1 : rd_off0));
      // an empty use here keeps the compiler from sinking each read into the
      // branch that multiplies it
#pragma unroll
      for (int i = 0; i < MW; ++i) asm volatile("" ::"v"(av[i]));
#pragma unroll
      for (int i = 0; i < MW; ++i) {
        if ((wr + RW * i) * 16 >= ti.rows) break;  // wave-uniform: row blocks past the tile
#pragma unroll
        for (int j = 0; j < Frag<T>::steps; ++j)
#pragma unroll
          for (int c = 0; c < 2 * CW; ++c) acc[i][c] = Frag<T>::mma(av[i], bf[c], j, acc[i][c]);
      }
      // the weight DMAs of stage kt + SB - 1 go out behind the first k half's
      // MFMAs, so their issue (the memory pipeline's back-pressure) overlaps the
      // matrix cores instead of delaying them; the issue order, and so every
      // vmcnt count, is unchanged (A of a step, then its B)
      if (h == 0 && kt + SB - 1 < NK) {
        const int s = kt + SB - 1;
        issue_b(ldsB + (s % SB) * P::BSZ, s);
      }
    }
    if (kt == nk - 1 && ntiles > 1) {
      store_tile(acc, nt0);
#pragma unroll
      for (int i = 0; i < MW; ++i)
#pragma unroll
        for (int c = 0; c < 2 * CW; ++c) acc[i][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  }
  store_tile(acc, nt0 + ntiles - 1);
}

// tile width in features (gate/up) or output columns (down) for CG column groups
template <bool GATEUP> constexpr int tile_width(int cg) { return GATEUP ? 16 * cg : 32 * cg; }

// OWN: a dense expert of another width is there (a kernel of its own: the selects of the
// width in the common one cost the matrix-bound tiles 3%).
// TPW (1 or 2): N tiles per workgroup, consecutive tiles of one M tile in one
// pipeline (gemm_tile).
// ROWS: the grid has several rows (launch_grouped; the row index in the common kernel cost
// fp32 layers of 65-200 tokens 0.2-0.8 us).
template <typename T, bool GATEUP, int CG, int W, int TPW, bool OWN, bool ROWS = false>
__global__ __launch_bounds__(W * 64) void grouped_gemm_kernel(GemmArgs a) {
  static_assert(TPW == 1 || TPW == 2, "one or two N tiles per workgroup");
  const int nN = (GATEUP ? a.m : a.d) / tile_width<GATEUP>(CG);
  const int block = static_cast<int>(ROWS ? (blockIdx.y << kPipeGridRow) + blockIdx.x : blockIdx.x);
  int grp, np, nt0, ntiles = 1;
  constexpr int TM = sizeof(T) == 4 ? kTileMF32 : kTileM;
  TileInfo ti;
  if (GATEUP && OWN && block >= a.sh_block0) {
    // the dense expert's tiles, of a width other than the routed experts'
    map_block(block - a.sh_block0, a.sh_m / tile_width<GATEUP>(CG), &grp, &nt0);
    ti.e = 0;
    ti.row0 = grp * TM;
    ti.rows = min(TM, a.sh_rows - ti.row0);
    ti.valid = ti.rows > 0;
    ti.sh = true;
    ti.once = a.sh_rows <= TM;
  } else {
    map_block(block, (nN + TPW - 1) / TPW, &grp, &np);
    nt0 = np * TPW;
    ntiles = min(TPW, nN - nt0);
    ti = tile_info<TM>(a, grp);
  }
  if (!ti.valid) return;
  __shared__ __align__(16) uint8_t smem[Pipe<16, CG, stage_halves<CG>(), W>::LDS];
  [[maybe_unused]] const int blocks = (ti.rows + 15) >> 4;
  // K rotation key: the expert (the appended dense expert gets its own)
  const int erot = ti.sh ? 0x155 : ti.e;
  if constexpr (sizeof(T) == 4) {  // tiles of at most 64 rows
    gemm_tile<T, GATEUP, kTileMF32 / 16, CG, stage_halves<CG>(), W, OWN>(a, ti, nt0, ntiles, erot, smem);
  } else {
    if (blocks <= 4)
      gemm_tile<T, GATEUP, 4, CG, stage_halves<CG>(), W, OWN>(a, ti, nt0, ntiles, erot, smem);
    else if (blocks <= 8)
      gemm_tile<T, GATEUP, 8, CG, stage_halves<CG>(), W, OWN>(a, ti, nt0, ntiles, erot, smem);
    else if (blocks <= 12)
      gemm_tile<T, GATEUP, 12, CG, stage_halves<CG>(), W, OWN>(a, ti, nt0, ntiles, erot, smem);
    else
      gemm_tile<T, GATEUP, 16, CG, stage_halves<CG>(), W, OWN>(a, ti, nt0, ntiles, erot, smem);
  }
}

// N tiles per workgroup.  Down: two (K is only m deep, so a tile is a short
// pipeline; the pair runs as one and the grid is one round of workgroups fewer:
// wider-pool down 153.9 -> 149.3 us, the 4096-token layer's unchanged).  Gate/up:
// one.  Two, three or four made it 9-50% slower, three even where its grid is
// exactly one round on the 256 CUs: with one tile per workgroup the N tiles of an
// M tile run at once on one XCD and share the gathered activation rows in its L2,
// while a workgroup walking its tiles one after the other gathers them again for
// each tile.
constexpr int kTpwGateUp = 1;
constexpr int kTpwDown = 2;
int pairs(int nN, int tpw) { return (nN + tpw - 1) / tpw; }

unsigned grid_for(int max_groups, int nN) {
  const int g8 = (max_groups + 7) / 8;
  return static_cast<unsigned>(8 * nN * g8);
}

// A launch takes fewer than 2^32 threads in x.  bf16 tiles are so large that the grid stays
// far below; fp32's 64-row tiles reach it at slots * m = 2^34 (an H of 64 GiB: 2^20 tokens,
// top-8, experts of 2048), where the grid gets several rows.
template <typename T, bool GATEUP, int CG, int TPW> void launch_grouped(const GemmArgs &a, hipStream_t stream) {
  const int nN = (GATEUP ? a.m : a.d) / tile_width<GATEUP>(CG);
  const unsigned grid = grid_for(a.max_groups, pairs(nN, TPW));
  GemmArgs b = a;
  unsigned blocks = grid;
  const bool own = a.sh_tiles > 0 && a.sh_m != a.m;
  if (own && GATEUP) {
    b.sh_tiles = 0;
    b.sh_block0 = static_cast<int>(grid);
    blocks += grid_for(a.sh_tiles, a.sh_m / tile_width<GATEUP>(CG));
  }
  const PipeGrid p = sizeof(T) == 4 ? pipe_grid(blocks, kGemmWaves * 64) : PipeGrid{blocks, 1};
  const dim3 dims(p.x, p.y);
  auto launch = [&](auto kernel) { kernel<<<dims, kGemmWaves * 64, 0, stream>>>(b); };
  if constexpr (sizeof(T) == 4)
    if (p.y > 1) {
      if (own)
        launch(grouped_gemm_kernel<T, GATEUP, CG, kGemmWaves, TPW, true, true>);
      else
        launch(grouped_gemm_kernel<T, GATEUP, CG, kGemmWaves, TPW, false, true>);
      return;
    }
  if (own)
    launch(grouped_gemm_kernel<T, GATEUP, CG, kGemmWaves, TPW, true>);
  else
    launch(grouped_gemm_kernel<T, GATEUP, CG, kGemmWaves, TPW, false>);
}

// column groups of the gate/up tiles for an intermediate size
int gateup_cg(int m, bool bf16) { return !bf16 ? 2 : m % tile_width<true>(8) == 0 ? 8 : 4; }

}  // namespace

bool gateup_takes_dense(int m, int sh_m, bool bf16) {
  return sh_m % tile_width<true>(gateup_cg(m, bf16)) == 0;
}

// bf16: 128 features per gate/up tile when they divide m, else 64; 256 output columns
// per down tile when they divide d, else 128.  fp32: 32 features, 64 columns.
hipError_t launch_gateup(const GemmArgs &a, bool bf16, hipStream_t stream) {
  if (a.max_groups <= 0) return hipSuccess;
  if (!bf16)
    launch_grouped<float, true, 2, 1>(a, stream);
  else if (gateup_cg(a.m, true) == 8)
    launch_grouped<bf16_t, true, 8, kTpwGateUp>(a, stream);
  else
    launch_grouped<bf16_t, true, 4, kTpwGateUp>(a, stream);
  return hipGetLastError();
}

hipError_t launch_down(const GemmArgs &a, bool bf16, hipStream_t stream) {
  if (a.max_groups <= 0) return hipSuccess;
  if (!bf16)
    launch_grouped<float, false, 2, 1>(a, stream);
  else if (a.d % tile_width<false>(8) == 0)
    launch_grouped<bf16_t, false, 8, kTpwDown>(a, stream);
  else
    launch_grouped<bf16_t, false, 4, kTpwDown>(a, stream);
  return hipGetLastError();
}

}  // namespace ace
