// Host side of the fp32 kernels: which products they take, tile choice, launches.
#include "fast32.hpp"

namespace ard {

// Sums the partial sums of a contraction split over the grid and writes the output through its (affine) maps:
// one thread per physical column, dropped positions included.
static __global__ void gemm_finish_f32_kernel(const float* part, int splits, int M, int N, OutMat C, FastDiv row_div, FastDiv col_div) {
  const int cols = C.fill ? C.cn.nphys : N, rows = C.fill ? C.rm.nphys : M;
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= cols) return;
  int j = c;
  bool col_kept = true;
  if (C.fill) {
    const int d = c - C.cn.off;
    j = d >= 0 ? (int)fdiv((uint32_t)d, col_div) : 0;
    col_kept = d >= 0 && j * C.cn.step == d && j < N;
  }
  for (int r = blockIdx.y; r < rows; r += gridDim.y) {
    int i = r;
    bool kept = col_kept;
    if (C.fill) {
      const int d = r - C.rm.off;
      i = d >= 0 ? (int)fdiv((uint32_t)d, row_div) : 0;
      kept = kept && d >= 0 && i * C.rm.step == d && i < M;
    }
    float x = 0.0f;
    if (kept)
      for (int s = 0; s < splits; ++s) x += part[((long)s * M + i) * N + j];
    const long idx = (long)(C.fill ? r : ax_phys(C.rm, r)) * C.ld + (C.fill ? c : ax_phys(C.cn, c));
    store_out<float>(C, idx, C.alpha * x, kept);
  }
}

// What a workgroup of a convolution costs: times its products at the matrix cores' rate, if it has a CU to itself and if two share
// it, and us to begin and to store its results.
struct F32ConvCost {
  float alone, pair, begin;
};
// Workgroup tiles: how the four wavefronts share it, contraction steps in flight, the share of the
// matrix-core rate a full chip of them reaches in products (128 x 128 on 2048^3, the small ones on products they fill), and
// costs in convolutions whose output rows are whole groups of four pixels (`fours`) or not (`ones`: pixels are fetched one by one).
struct F32Cfg {
  int bm, bn, wk, d;
  float eff;
  F32ConvCost fours, ones;
};
// The last four are for convolutions alone: few channels, any number of pixels, whose wavefronts lie side by side along the
// pixels so that a contraction of a few dozen steps is not dealt over them as well (64 rows, 65536 pixels, 18 steps:
// 32 us against 43 with 64 x 64 tiles; 32 rows, 36 steps: 29 against 43 with 32 x 32 tiles; 64 rows, 25088 pixels, 72 steps,
// layer 71 us with 32 x 32 tiles, 57 with 32 x 256, 60 with 64 x 128).
static const F32Cfg kF32Cfgs[8] = {{128, 128, 1, 3, 0.85f, {1.15f, 1.82f, 4.39f}, {1.17f, 2.51f, 8.88f}},
                                   {64, 64, 4, 3, 0.8f, {1.08f, 1.57f, 4.31f}, {1.1f, 1.9f, 6.69f}},
                                   {32, 32, 4, 4, 0.6f, {1.7f, 1.9f, 1.58f}, {2.23f, 2.25f, 1.62f}},
                                   {16, 16, 4, 8, 0.4f, {3.03f, 3.08f, 0.99f}, {4.24f, 3.83f, 1.11f}},
                                   {64, 256, 1, 3, 0.0f, {0.96f, 1.65f, 4.63f}, {1.1f, 2.77f, 10.48f}},
                                   {32, 256, 1, 4, 0.0f, {1.13f, 1.83f, 1.9f}, {1.7f, 2.95f, 4.81f}},
                                   {64, 128, 1, 3, 0.0f, {1.3f, 2.09f, 3.16f}, {1.22f, 2.71f, 3.38f}},
                                   {32, 128, 1, 4, 0.0f, {1.48f, 1.82f, 1.77f}, {2.03f, 2.31f, 1.69f}}};

// Do the results of a 32 x 32 tile leave in runs of four physical columns (one store each, zeros of the dropped ones included)?  Where
// columns lie three and more apart, or two and rows are dropped as well: 260 weight gradients of up to 1024 rows, 3072 x 4096 neurons, 0.97
// of the time in the mean, 0.57 at best (128 x 2048 -> 2048, dp 3 and 3 12.8 -> 11.1 us, 5 and 5 16.6 -> 12.7); 220 forward products and data
// gradients without compact layouts 0.99, 0.72 at best.  Every second column of whole rows: 1.01 and 1.00 in the mean (55 x 254 -> 2688, dp 1
// and 2 6.95 -> 7.18 us), every column 19.5 -> 20.0 (128 x 2048 -> 2048, dp 2 and 1).
static bool f32_leaves_in_runs(const F32Params& F) {
  const OutMat& C = F.C;
  return !F.part && F.tab.ncls == 0 && C.fill && C.beta == 0.0f && C.cn.kind == AX_AFFINE && (C.cn.step > 2 || (C.cn.step == 2 && C.rm.kind == AX_AFFINE && C.rm.step > 1));
}

template <int AK, int BK, int MODE>
static int32_t launch_f32(F32Params& F, int cfg, int grid, hipStream_t stream) {
  const F32Cfg& c = kF32Cfgs[cfg];
  const size_t lds = (size_t)c.wk * c.bm * (c.bn + 1) * 4 + (size_t)(c.bm * 3 > c.bm + c.bn ? c.bm * 3 : c.bm + c.bn) * 4;  // accumulators, tables
  const dim3 g((unsigned)grid), b(256);
#define ARD_F32_CASE(I, ...) ARD_F32_INSTANCE(I, false, __VA_ARGS__)
#define ARD_F32_INSTANCE(I, IN_RUNS, ...)                                                                \
  case I: {                                                                                              \
    auto kernel = gemm_f32_kernel<AK, BK, __VA_ARGS__, MODE, IN_RUNS>;                                   \
    static thread_local bool raised = false;                                                             \
    if (!raised && lds >= 65536) {                                                                       \
      ARD_HIP_CHECK(raise_lds_limit((const void*)kernel, (int)lds));                                     \
      raised = !dry_run();                                                                               \
    }                                                                                                    \
    ARD_LAUNCH_NAMED(launch_instance(IN_RUNS ? "gemm_f32_kernel<runs>" : "gemm_f32_kernel", c.bm, c.bn, MODE), kernel, g, b, lds, stream, F); \
    break;                                                                                               \
  }
  if constexpr (MODE == 1) {
    switch (cfg) {
      ARD_F32_CASE(4, 4, 4, 1, 4, 1, 3)
      ARD_F32_CASE(5, 2, 4, 1, 4, 1, 4)
      ARD_F32_CASE(6, 4, 2, 1, 4, 1, 3)
      ARD_F32_CASE(7, 2, 2, 1, 4, 1, 4)
      default: break;
    }
  }
  const bool in_runs = MODE == 0 && cfg == 2 && f32_leaves_in_runs(F);
  if constexpr (MODE == 0) {
    if (in_runs) switch (cfg) {
      ARD_F32_INSTANCE(2, true, 2, 2, 1, 1, 4, 4)
    }
  }
  if (!in_runs) switch (cfg) {
    ARD_F32_CASE(0, 4, 4, 2, 2, 1, 3)
    ARD_F32_CASE(1, 4, 4, 1, 1, 4, 3)
    ARD_F32_CASE(2, 2, 2, 1, 1, 4, 4)
    ARD_F32_CASE(3, 1, 1, 1, 1, 4, 8)
    case 4: case 5: case 6: case 7: break;
    default: return fail(ARD_EUNSUPPORTED, "no such fp32 tile");
  }
#undef ARD_F32_CASE
#undef ARD_F32_INSTANCE
  ARD_LAUNCH_CHECK("gemm_f32_kernel");
  return ARD_OK;
}

static int32_t launch_f32_kinds(int ak, int bk, F32Params& F, int cfg, int grid, hipStream_t stream) {
#define ARD_F32_KINDS(A, B) \
  if (ak == A && bk == B) return launch_f32<A, B, 0>(F, cfg, grid, stream);
  ARD_F32_KINDS(F32_KC_VEC, F32_KC_VEC)
  ARD_F32_KINDS(F32_KC_VEC, F32_KC)
  ARD_F32_KINDS(F32_KC, F32_KC_VEC)
  ARD_F32_KINDS(F32_KC, F32_KC)
  ARD_F32_KINDS(F32_KC_VEC, F32_MC_VEC)
  ARD_F32_KINDS(F32_KC_VEC, F32_MC)
  ARD_F32_KINDS(F32_KC, F32_MC_VEC)
  ARD_F32_KINDS(F32_KC, F32_MC)
  ARD_F32_KINDS(F32_MC_VEC, F32_MC_VEC)
  ARD_F32_KINDS(F32_MC_VEC, F32_MC)
  ARD_F32_KINDS(F32_MC, F32_MC_VEC)
  ARD_F32_KINDS(F32_MC, F32_MC)
#undef ARD_F32_KINDS
  return fail(ARD_EUNSUPPORTED, "operand layout combination not built");
}

// Time of a product with this tile, in clocks: rounds of workgroups over 256 CUs (the wavefronts of several
// workgroups on a CU share its matrix cores, 256 FLOP per clock) against the chain of memory round trips of
// one wavefront (about 1500 clocks per D steps), and what it takes to store the `spread` physical positions
// per result (zeros of dropped rows and columns included): about 4 per clock and CU, and 600 clocks for a
// workgroup to come and go.
static float f32_clocks(const F32Cfg& c, long tiles, int K, int splits, float spread) {
  const float rounds = (float)((tiles * splits + 255) / 256);
  const float k = (float)K / splits;
  const float mfma = rounds * c.bm * c.bn * k * (2.0f / 256.0f) / c.eff;
  const int steps = imax(1, (int)(k / 16.0f / c.wk));
  const float chain = 1500.0f * ((steps + c.d - 1) / c.d);
  return (mfma > chain ? mfma : chain) + rounds * (600.0f + 0.25f * c.bm * c.bn * (splits > 1 ? 1.0f : spread));
}

static bool affine(const Axis& a) { return a.kind == AX_AFFINE && a.step >= 1 && a.off >= 0; }
bool f32_takes_maps(const Axis& out, const Axis& in) {
  return !dev_knobs().no_fast && affine(in) && affine(out);
}

bool try_f32(bool a_kc, bool b_kc, const GemmParams& P, void* ws, size_t ws_bytes, hipStream_t stream, int32_t& st) {
  if (dev_knobs().no_fast || P.kb_ptr || P.tmask || P.C.plane || (!a_kc && b_kc)) return false;
  if (P.M < 1 || P.N < 1 || (long)P.M * P.N >= (1L << 31) || P.k.n < 0) return false;
  const Axis ka = P.A.kdense ? axis_identity(P.k.n) : P.k, kb = P.B.kdense ? axis_identity(P.k.n) : P.k;
  if (!affine(ka) || !affine(kb)) return false;
  for (const Operand* op : {&P.A, &P.B}) {
    const bool kc = op == &P.A ? a_kc : b_kc;
    const Axis& k = op == &P.A ? ka : kb;
    if (!(affine(op->r) || op->r.kind == AX_LIST) || op->r.n < 1) return false;
    if (k.n > 0 && k.off + (long)(k.n - 1) * k.step >= k.nphys) return false;
    if (affine(op->r) && op->r.off + (long)(op->r.n - 1) * op->r.step >= op->r.nphys) return false;
    if (((uintptr_t)op->p & 3) || (long)imax(kc ? op->r.nphys : k.nphys, 1) * op->ld * 4 >= (1L << 31)) return false;
  }
  auto kind = [](bool kc, const Axis& r, const Axis& k) {
    if (kc) return k.step == 1 ? (int)F32_KC_VEC : (int)F32_KC;
    return r.kind == AX_AFFINE && r.step == 1 && r.n >= 4 ? (int)F32_MC_VEC : (int)F32_MC;
  };
  const OutMat& C = P.C;
  auto owned = [](const Axis& a) { return a.kind == AX_AFFINE && a.off < a.step; };
  auto map_ok = [&](const Axis& a) { return a.kind == AX_LIST || (C.fill ? owned(a) : a.kind == AX_AFFINE); };
  if (!map_ok(C.rm) || !map_ok(C.cn)) return false;
  F32Params F{};
  F.A = (const float*)P.A.p, F.B = (const float*)P.B.p;
  F.lda = (int)P.A.ld, F.ldb = (int)P.B.ld;
  F.am = P.A.r, F.bn = P.B.r, F.k = axis_identity(P.k.n);
  F.ka_off = ka.off, F.ka_step = ka.step, F.kb_off = kb.off, F.kb_step = kb.step;
  F.C = C;
  F.row_div = fast_div((uint32_t)C.rm.step), F.col_div = fast_div((uint32_t)C.cn.step);
  F.M = P.M, F.N = P.N;
  // Tile, and whether the contraction is split over the grid as well: a finishing pass costs about 12000
  // clocks (a dependent launch that reads what other XCDs wrote).
  const bool can_split = ws && C.rm.kind == AX_AFFINE && C.cn.kind == AX_AFFINE;
  const float spread = C.fill ? (float)((double)C.rm.nphys * C.cn.nphys / ((double)P.M * P.N)) : 1.0f;
  int cfg = 0, splits = 1;
  float best = 0.0f;
  for (int i = 0; i < 4; ++i) {
    const F32Cfg& c = kF32Cfgs[i];
    const long tiles = (long)ceil_div(P.M, c.bm) * ceil_div(P.N, c.bn);
    if (tiles >= (1L << 24)) continue;
    for (int sp = 1; sp <= 16; sp *= 2) {
      if (sp > 1 && (!can_split || P.k.n < 16 * c.wk * c.d * sp || (size_t)sp * P.M * P.N * 4 > ws_bytes)) break;
      const float t = f32_clocks(c, tiles, P.k.n, sp, spread) + (sp > 1 ? 12000.0f : 0.0f);
      if (best == 0.0f || t < best) best = t, cfg = i, splits = sp;
    }
  }
  if (best == 0.0f) return false;
  const F32Cfg& c = kF32Cfgs[cfg];
  F.tiles_m = ceil_div(P.M, c.bm), F.tiles_n = ceil_div(P.N, c.bn);
  F.total_tiles = F.tiles_m * F.tiles_n;
  set_bands(F, direct_group_m(F.total_tiles));
  F.splits = splits;
  if (splits > 1) F.part = (float*)ws;
  st = launch_f32_kinds(kind(a_kc, F.am, ka), kind(b_kc, F.bn, kb), F, cfg, direct_plain_grid(F.total_tiles * splits), stream);
  if (st || splits == 1) return true;
  const int cols = C.fill ? C.cn.nphys : P.N, rows = C.fill ? C.rm.nphys : P.M;
  ARD_LAUNCH(gemm_finish_f32_kernel, dim3((unsigned)ceil_div(cols, 256), (unsigned)imin(rows, 4096)), dim3(256), 0, stream,
             (const float*)F.part, splits, P.M, P.N, C, F.row_div, F.col_div);
  const hipError_t e = launch_status();
  if (e != hipSuccess) st = fail(ARD_EHIP, "launch of gemm_finish_f32_kernel failed: %s", hipGetErrorString(e));
  return true;
}

// Convolution on the zero-bordered channel planes of the grid (conv.hip): C[row][pixel] = sum over (tap, channel)
// of W[row][tap*Cp + channel] * grid, row r stored to channel plane C.rm(r).
int32_t f32_conv_product(const float* W, int rows, const float* grid, const F32Conv& cv, const OutMat& C, hipStream_t stream) {
  F32Params F{};
  const int taps_cp = cv.taps * cv.Cp;
  F.A = W, F.B = grid, F.lda = taps_cp;
  F.am = axis_identity(rows), F.bn = axis_identity(cv.npix), F.k = axis_identity(taps_cp);
  F.C = C, F.M = rows, F.N = cv.npix, F.splits = 1;
  F.cv = cv;
  // Tile of the least estimated time.  Workgroups come two to a CU; up to four a CU the last pair, or single one, counts in full, beyond
  // it starts here and there as others end.  Costs fitted to the products of 870 layers, forward and data gradient (610 of 8 - 128
  // images, 16 - 512 channels, 7 x 7 - 56 x 56, filters of 1, 3 and 5, a third to all maps kept; 260 of up to 40 images and 12000
  // pixels, contractions of up to 12800).  In 305 and 260 others the choice is 1.3 and 0.7 % off the best tile in the mean, 9 and 5 %
  // at the 95th percentile (one share of the matrix-core rate per tile and whole rounds: 4.1 and 1.5, 23 and 11 %).  21 images, 48 ->
  // 192 channels of 56 x 56: 64 x 64 tiles 147 us, 64 x 256 170; 8 images of 16 x 16, 33 of 110 channels <- 248, 5 x 5, data
  // gradient: 16 x 16 tiles 5 us less than 32 x 32.
  const bool fours = cv.Wo % 4 == 0;
  int cfg = 0;
  float best = 0.0f;
  for (int i = 0; i < 8; ++i) {
    const F32Cfg& c = kF32Cfgs[i];
    const F32ConvCost& w = fours ? c.fours : c.ones;
    const long tiles = (long)ceil_div(rows, c.bm) * ceil_div(cv.npix, c.bn), whole = (tiles + 255) / 256;  // on the fullest CU
    const float product = (float)c.bm * c.bn * taps_cp * (2.0f / (256.0f * 2400.0f)), two = 2.0f * w.pair * product + w.begin;  // us at 2.4 GHz
    const float t = whole > 4 ? two * 0.25f * (tiles / 256.0f + whole) : two * (whole / 2) + (whole % 2 ? w.alone * product + w.begin : 0.0f);
    if (i == 0 || t < best) best = t, cfg = i;
  }
  F.tiles_m = ceil_div(rows, kF32Cfgs[cfg].bm), F.tiles_n = ceil_div(cv.npix, kF32Cfgs[cfg].bn);
  if ((long)F.tiles_m * F.tiles_n >= (1L << 24)) return fail(ARD_ESHAPE, "convolution too large for one launch");
  F.total_tiles = F.tiles_m * F.tiles_n;
  set_bands(F, direct_group_m(F.total_tiles));
  const int grid_x = direct_plain_grid(F.total_tiles);
  // (groups of four pixels are contiguous where output rows are whole numbers of them)
  return fours ? launch_f32<F32_KC_VEC, F32_MC_VEC, 1>(F, cfg, grid_x, stream) : launch_f32<F32_KC_VEC, F32_MC, 1>(F, cfg, grid_x, stream);
}

// Its weight gradient: part[split][co][tap*Cp + channel] = sum over the pixels of the grid planes of dY * A, both
// read along their planes; the contraction is split until the chip is full, `cap` partial results at most.
// Returns the number of splits through *splits.
int32_t f32_conv_wgrad(const float* grid_y, const float* grid_a, const F32Conv& cv, int N, int rows, int cap, float* part, int* splits,
                       hipStream_t stream) {
  F32Params F{};
  const int cols = cv.taps * cv.Cp, K = N * cv.plane, steps = K / 16;
  F.A = grid_y, F.B = grid_a, F.lda = cv.plane;
  F.am = axis_identity(rows), F.bn = axis_identity(cols), F.k = axis_identity(K);
  F.M = rows, F.N = cols;
  F.cv = cv;
  F.part = part;
  int cfg = 1, sp = 1;
  float best = 0.0f;
  for (int i = 0; i < 3; ++i) {
    const F32Cfg& c = kF32Cfgs[i];
    const long tiles = (long)ceil_div(rows, c.bm) * ceil_div(cols, c.bn);
    for (int s = 1; s <= cap && s * 4 * c.wk <= imax(steps, 4 * c.wk); s = s < 8 ? s + 1 : s + s / 4) {
      // (what the pass over the partial results costs: they come and go at about 1000 bytes a clock)
      const float t = f32_clocks(c, tiles, K, s, 1.0f) + (float)s * rows * cols * 8.0f / 1000.0f;
      if (best == 0.0f || t < best) best = t, cfg = i, sp = s;
    }
  }
  F.tiles_m = ceil_div(rows, kF32Cfgs[cfg].bm), F.tiles_n = ceil_div(cols, kF32Cfgs[cfg].bn);
  if ((long)F.tiles_m * F.tiles_n * sp >= (1L << 24)) return fail(ARD_ESHAPE, "convolution too large for one launch");
  F.total_tiles = F.tiles_m * F.tiles_n;
  F.splits = sp;
  set_bands(F, direct_group_m(F.total_tiles));
  *splits = sp;
  return launch_f32<F32_KC_VEC, F32_KC_VEC, 2>(F, cfg, direct_plain_grid(F.total_tiles * sp), stream);
}

// Tile pattern (Section 3.2): classes of tile rows or columns as in the bf16 kernels (tile_classes); any tile
// size works, a tile wider than the workgroup's tile is taken in parts.
bool try_f32_tile(int op, int B, int I, int O, int TR, int TC, const ard_pattern& pat, const void* Ap, const void* Bp, void* Cp,
                  float alpha, int relu, const void* relu_src, hipStream_t stream, int32_t& st) {
  if (dev_knobs().no_fast) return false;
  if ((long)B * O * 4 >= (1L << 31) || (long)B * I * 4 >= (1L << 31) || (long)O * I * 4 >= (1L << 31)) return false;
  if (((uintptr_t)Ap & 3) || ((uintptr_t)Bp & 3)) return false;
  const int x = pat.tile_r, y = pat.tile_c, dp = pat.dp, o = pat.b - 1;
  F32Params F{};
  ClassTab& t = F.tab;
  if (!tile_classes(op, O, I, TR, TC, x, y, dp, o, t)) return false;
  F.A = (const float*)Ap, F.B = (const float*)Bp;
  F.ldb = I;
  F.ka_step = F.kb_step = 1;
  F.c_cols_mapped = 1;
  F.C.p = Cp, F.C.alpha = alpha, F.C.relu = relu, F.C.relu_src = relu_src;
  int ak = F32_KC_VEC, bk = F32_KC_VEC;
  if (op == 0) {
    F.lda = I, F.am = axis_identity(B), F.C.ld = O, F.M = B, F.N = O;
  } else {
    // (groups of four columns must not straddle the end of the matrix: a block progression is not moved back)
    bk = I % 4 == 0 ? F32_MC_VEC : F32_MC;
    F.lda = O, F.C.ld = I, F.N = I;
    if (op == 1) {
      F.am = axis_identity(B), F.M = B;
    } else {
      ak = O % 4 == 0 ? F32_MC_VEC : F32_MC;
      F.k = axis_identity(B), F.c_rows_mapped = 1, F.M = O;
    }
  }
  int K = op == 2 ? B : 0, heavy = 0, cfg = -1;
  if (op != 2)
    for (int c = 0; c < t.ncls; ++c) K = imax(K, t.k_cnt[c] * t.k_bs);
  float best = 0.0f;
  for (int i = 0; i < 4; ++i) {
    const F32Cfg& c = kF32Cfgs[i];
    if (!tile_run_fits(t.n_bs, c.bn) || (op == 2 && !tile_run_fits(t.m_bs, c.bm))) continue;
    if (count_classes(op, t, B, c.bm, c.bn, heavy) == 0) continue;
    const float est = f32_clocks(c, imax(heavy, 1), K, 1, 1.0f);
    if (cfg < 0 || est < best) best = est, cfg = i;
  }
  if (cfg < 0) return false;
  F.total_tiles = count_classes(op, t, B, kF32Cfgs[cfg].bm, kF32Cfgs[cfg].bn, heavy);
  set_bands(F, direct_group_m(F.total_tiles));
  F.splits = 1;
  if (op == 2) {
    ARD_LAUNCH(zero_dropped_tiles_kernel<float>, dim3((unsigned)(TR * TC)), dim3(256), 0, stream, (float*)Cp, I, O, I, x, y, TC, dp, o);
    const hipError_t e = launch_status();
    if (e != hipSuccess) {
      st = fail(ARD_EHIP, "launch of zero_dropped_tiles_kernel failed: %s", hipGetErrorString(e));
      return true;
    }
  }
  st = launch_f32_kinds(ak, bk, F, cfg, class_grid(F.tab), stream);
  return true;
}

}  // namespace ard
