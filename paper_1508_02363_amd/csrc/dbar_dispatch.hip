// Run-time dispatch over the grid size N for the line-transform stages.
#include <algorithm>
#include <atomic>

#include "dbar_lines.h"

namespace dbar {

// ------------------------------------------------------------------------------------------------------------
// Column-tile width choices (set by the tuner; default 0 = the narrowest tile)
// ------------------------------------------------------------------------------------------------------------
static int size_index(int N) {
  int i = 0;
  for (int m = 8; m < N && i < 12; m <<= 1) ++i;
  return i;
}
static std::atomic<int> g_tile[2][12];  // [fp64][log2(N) - 3]
static std::atomic<int> g_epoch{0};

int tile_variants(int N, bool fp64) {
#define DBAR_VARIANTS(NN) \
  if (N == NN) return fp64 ? Tiling<double, NN>::variants() : Tiling<float, NN>::variants();
  DBAR_FOR_EACH_N(DBAR_VARIANTS)
#undef DBAR_VARIANTS
  return 1;
}

int tile_variant(int N, bool fp64) { return g_tile[fp64 ? 1 : 0][size_index(N)].load(); }

void set_tile_variant(int N, bool fp64, int variant) {
  if (variant < 0 || variant >= tile_variants(N, fp64)) variant = 0;
  if (g_tile[fp64 ? 1 : 0][size_index(N)].exchange(variant) != variant) ++g_epoch;
}

int tuning_epoch() { return g_epoch.load(); }

template <typename T, int N>
static int tile_cols(int variant) {
  using Tl = Tiling<T, N>;
  switch (variant) {
    case 1: return Tl::template cols_v<1>();
    case 2: return Tl::template cols_v<2>();
    case 3: return Tl::template cols_v<3>();
    default: return Tl::COLS;
  }
}

// tiles of the column stage that leaves moment partials (its threads may limit its columns below the variant's)
template <typename T, int N>
static int moment_cols(int variant) {
  using Tl = Tiling<T, N>;
  constexpr int E = Ept<T, N>::MOMENT_COLS;
  switch (variant) {
    case 1: return Tl::template cols_of<E, 1, true>();
    case 2: return Tl::template cols_of<E, 2, true>();
    case 3: return Tl::template cols_of<E, 3, true>();
    default: return Tl::template cols_of<E, 0, true>();
  }
}

int moment_tiles(int N, bool fp64) {
  const int v = tile_variant(N, fp64);
#define DBAR_TILES(NN) \
  if (N == NN) return NN / (fp64 ? moment_cols<double, NN>(v) : moment_cols<float, NN>(v));
  DBAR_FOR_EACH_N(DBAR_TILES)
#undef DBAR_TILES
  return 0;
}

int line_tiles_variant(int N, bool cols, bool fp64, int variant) {
#define DBAR_TILES(NN)                                                                               \
  if (N == NN) {                                                                                     \
    if (fp64) return NN / (cols ? tile_cols<double, NN>(variant) : Tiling<double, NN>::ROWS);        \
    return NN / (cols ? tile_cols<float, NN>(variant) : Tiling<float, NN>::ROWS);                    \
  }
  DBAR_FOR_EACH_N(DBAR_TILES)
#undef DBAR_TILES
  return 0;
}

int line_tiles_max(int N, bool cols, bool fp64) {
  int t = 0;
  for (int v = 0; v < (cols ? tile_variants(N, fp64) : 1); ++v) t = std::max(t, line_tiles_variant(N, cols, fp64, v));
  return t;
}

int tile_columns(int N, bool fp64, int variant) { return N / line_tiles_variant(N, true, fp64, variant); }

int line_tiles(int N, bool cols, bool fp64) {
  return line_tiles_variant(N, cols, fp64, cols ? tile_variant(N, fp64) : 0);
}

size_t tail_table_size(int N) { return (size_t)tail_pitch(N) * tail_pitch(N); }

__global__ void __launch_bounds__(256) k_tail_table(int N, double L, int M, c64* t64, c32* t32) {
  const int n = tail_pitch(N) * tail_pitch(N);
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) tail_table_entry(i, N, L, M, t64, t32);
}
bool launch_tail_table(int N, double L, int M, c64* t64, c32* t32, hipStream_t s) {
  const size_t n = tail_table_size(N);
  TimerScope ts(kStageControl, 0.0, 1, nullptr, s);
  void* args[] = {&N, &L, &M, &t64, &t32};
  if (hipLaunchKernel(reinterpret_cast<const void*>(k_tail_table), dim3((unsigned)((n + 255) / 256)), dim3(256), args, 0,
                      s) == hipSuccess)
    return true;
  (void)hipGetLastError();
  return false;
}

int box_row_align(int N) {
  return std::max(kBoxCols, std::max(N / line_tiles(N, false, true), N / line_tiles(N, false, false)));
}

// Algorithmic HBM bytes of one stage (each array read or written once): per batch entry, and once per launch for the
// potential when all entries share it (Q_bs = 0: one array read at stride 0 by every entry).
static double line_bytes_once(int N, LineOp op, const LineArgs& a, size_t es) {
  const bool reads_q = op == LineOp::ColsInvTailFwd || op == LineOp::RowsInvTailEpilogue ||
                       op == LineOp::ColsFwdPotential;
  const double in = op == LineOp::RowsInvTailEpilogue ? a.box_fr * a.box_fc : 1.0;
  return reads_q && a.Q_bs == 0 ? in * N * N * es : 0.0;
}
static double line_bytes(int N, LineOp op, const LineArgs& a, size_t es) {
  const double P = (double)N * N * es;
  const double PQ = a.Q_bs == 0 ? 0.0 : P;  // the potential, when every entry reads its own
  switch (op) {
    case LineOp::RowsInvScaled: return 2 * P;
    case LineOp::ColsInvMoments: return P;
    case LineOp::RowsInvRegular: return 2 * P;
    case LineOp::ColsInvTailFwd: return 2 * P + PQ + (a.hout ? P : 0.0);
    case LineOp::ColsInvTail: return 2 * P;
    case LineOp::RowsFwdEpilogue:  // fused dots read V_i, i < dot_nv - 1, besides S (= V_{dot_nv - 1})
      return 2 * P + (a.alpha != 0.0 ? P : 0.0) + (a.gamma != 0.0 ? P : 0.0) +
             (a.dot_nv > 0 ? (a.dot_nv - (a.alpha != 0.0 ? 1 : 0)) * P : 0.0);
    case LineOp::ColsFwdPotential: return P + PQ;
    case LineOp::ColsFwdPlain: return 2 * P;
    case LineOp::ColsInvPlain: return 2 * P;
    // x-space stages: s, the basis, Q and the result live on the box, the transform array on its rows (all rows where h
    // is wanted on the whole grid)
    case LineOp::RowsFwdMoments:
      return a.box_fr * (P + a.box_fc * (P + (a.upd_coef ? P + a.upd_nv * (a.upd_v32 ? P / 2 : P) : 0.0)));
    case LineOp::ColsFwdRegularInv: return (a.box_fr + (a.box_full ? 1.0 : a.box_fr)) * P + (a.sout ? P : 0.0);
    case LineOp::RowsInvTailEpilogue:  // in, Q (per entry unless shared), out, S, Y (unless formed from q_k), h, the
                                       // FP32 copy, earlier basis
      return (a.box_full ? 1.0 : a.box_fr) * P + (a.hout ? P : 0.0) +
             a.box_fr * a.box_fc *
                 (PQ + (a.out ? P : 0.0) + (a.out32 ? P / 2 : 0.0) + (a.alpha != 0.0 ? P : 0.0) +
                  (a.gamma != 0.0 && !a.y_rhs ? P : 0.0) +
                  (a.dot_nv > 0 ? (a.dot_nv - (a.alpha != 0.0 ? 1 : 0)) * P : 0.0));
  }
  return 0.0;
}

template <typename T>
void launch_lines_any(int N, LineOp op, const LineArgs& a_in, hipStream_t s) {
  TimerScope ts(kStageLines + 2 * static_cast<int>(op) + (sizeof(T) == 4 ? 1 : 0),
                line_bytes(N, op, a_in, sizeof(cx<T>)), a_in.B, a_in.act, s, line_bytes_once(N, op, a_in, sizeof(cx<T>)));
  LineArgs a = a_in;
  a.tile = tile_variant(N, sizeof(T) == 8);
  switch (N) {
#define DBAR_CASE(NN) \
  case NN:            \
    launch_lines<T, NN>(op, a, s); \
    break;
    DBAR_FOR_EACH_N(DBAR_CASE)
#undef DBAR_CASE
    default:
      break;
  }
}

template void launch_lines_any<double>(int, LineOp, const LineArgs&, hipStream_t);
template void launch_lines_any<float>(int, LineOp, const LineArgs&, hipStream_t);

}  // namespace dbar
