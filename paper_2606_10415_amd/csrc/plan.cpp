// Host-side launch planning of liblt (no device code): which GEMM launches
// take a split-K last wave and how much workspace that needs.  Compiled into
// the library with the kernels, and on its own into the host-only sanitizer
// check of the C ABI.
#include "kernels.hpp"

namespace lt {

// The split a workspace is sized for.  gemm_plan below decides whether a call
// with a workspace takes it; the size keeps room for it either way.
bool gemm_splitk_tail(int64_t M, int64_t N, int64_t K, SplitTail* p) {
  // the geometry of the half-tile tail (256x256 tiles, one wave = 256 CUs),
  // with the last wave's K split so that its units fill about one wave; a
  // launch of less than about one wave of 256x256 tiles is split whole
  // (split_at = 0: no full-K part) when that beats 128x128 tiles with full
  // K: the split gives twice their workgroups (S = 8) or each split still
  // runs a long K loop (K / S >= kLongK); otherwise the workspace round trip
  // costs more than the larger tile saves
  constexpr int64_t kCUs = 256, kMinSlices = 8, kMaxSplits = 8, kLongK = 2048;
  if (M <= 0 || N <= 0 || K <= 0) return false;
  // the partial tiles and their sum move 8 columns at a time, and a ragged K
  // takes its own launch: both need multiples of 8
  if ((N & 7) || (K & 7)) return false;
  // beyond the sizes the GEMM entry points accept: no plan (and no overflow)
  if (M > ((int64_t)1 << 30) || N > ((int64_t)1 << 30) || K > ((int64_t)1 << 30)) return false;
  const int64_t tm = (M + 255) / 256, tn = (N + 255) / 256, tiles = tm * tn;
  const int64_t nk = (K + 63) / 64;
  if (tiles < 192) {
    int64_t S = kCUs / tiles;
    if (S > kMaxSplits) S = kMaxSplits;
    if (S > nk / kMinSlices) S = nk / kMinSlices;
    if (S < 2) return false;
    if (S < kMaxSplits && K < kLongK * S) return false;
    p->columns = true;
    p->split_at = 0;
    p->Mt = M;
    p->Nt = N;
    p->S = (int)S;
    return true;
  }
  const int64_t waves = tiles / kCUs, rem = tiles % kCUs;
  if (waves < 1 || rem == 0 || 2 * rem > kCUs) return false;
  int64_t S = kCUs / rem;
  if (S > kMaxSplits) S = kMaxSplits;
  if (S > nk / kMinSlices) S = nk / kMinSlices;
  if (S < 2) return false;
  const int64_t full = waves * kCUs;
  if (full % tm == 0 && full / tm < tn) {
    p->columns = true;
    p->split_at = (full / tm) * 256;
    p->Mt = M;
    p->Nt = N - p->split_at;
  } else if (full % tn == 0 && full / tn < tm) {
    p->columns = false;
    p->split_at = (full / tn) * 256;
    p->Mt = M - p->split_at;
    p->Nt = N;
  } else {
    return false;
  }
  p->S = (int)S;
  return true;
}

size_t gemm_splitk_ws_bytes(int64_t M, int64_t N, int64_t K) {
  SplitTail p;
  if (!gemm_splitk_tail(M, N, K, &p)) return 0;
  return (size_t)p.S * (size_t)p.Mt * (size_t)p.Nt * sizeof(float);
}

namespace {

constexpr int64_t kPlanCUs = 256;
// Time of one 64-wide K-slice of a tile (us; NT / NN and TN layouts), what it
// adds with every CU busy (power lowers the clock, operand loads share L2 and
// the memory-side cache), and the rest of a round of tiles (prologue,
// epilogue and its memory traffic) for the plain, gate/up and SwiGLU-gradient
// epilogues and, in the plain one, for reading R.  Fitted to calls whose
// operands come from HBM, as a program's weights and activations do (calls
// on cached operands run 10-25% faster, the smaller tiles most): 1024 x 4096 x
// {4096, 11008} NT take 96 / 257 us as 256x256 tiles, 57 / 154 as 256x128,
// 42 / 110 as 128x128, 77 / 194 as 64x64; 4096 x 4096 x {4096, 11008} 109 / 285,
// 123 / 321, 154 / 411, 297 / 745.
// Leading dimensions that are no multiple of 64 elements (`split_rows`): the
// 128 bytes that a slice reads of each row then lie in two memory lines.  The
// larger tiles hide that behind their MFMAs; the 64x64 tile's slices take
// 1.2 (TN 1.3) times as long, the 128x128 tile's 1.07.  Over 880 random
// shapes with K from 64 to 16384, 626 of them with a split-K plan: without
// these factors 70 ran as whole-K tiles more than 10% slower than split (128 x
// 5160 x 10616 NT 88 us against 54), with them 19, the worst 1.26 times.
struct TileCost {
  double slice, slice_tn, load, fixed[3], r, split_rows, split_rows_tn;
};
constexpr TileCost kTileCost[kNumGemmTiles] = {
    {1.48, 1.42, 0.10, {4.0, 6.0, 18.0}, 6.0, 1.0, 1.0},
    {0.87, 0.92, 0.03, {3.0, 4.5, 11.0}, 3.0, 1.0, 1.0},
    {0.87, 0.92, 0.03, {3.0, 4.5, 13.0}, 3.0, 1.0, 1.0},
    {0.50, 0.55, 0.10, {1.5, 2.0, 6.0}, 1.5, 1.07, 1.0},
    {0.25, 0.26, 0.02, {1.5, 3.0, 5.5}, 0.5, 1.2, 1.3},
};
constexpr double kLaunchUs = 4.0;             // a further launch in the stream
// split-K partials, written, then read: above the memory's rate, as the 64 MiB
// at most of them stay in the 256 MiB memory-side cache
constexpr double kPartialBytesPerUs = 9.0e6;

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// what one call's tiles have in common
struct TileKind {
  bool tn, split_rows;
  int epi;
};

// us of `tiles` tiles of a kind, nk K-slices each
double tiles_cost(int tile, const TileKind& k, bool reads_r, int64_t tiles, int64_t nk) {
  const TileCost& c = kTileCost[tile];
  const double slice = (k.tn ? c.slice_tn : c.slice) * (!k.split_rows ? 1.0 : k.tn ? c.split_rows_tn : c.split_rows);
  auto round = [&](int64_t n) {
    return (double)nk * (slice + c.load * (double)n / kPlanCUs) + c.fixed[k.epi] + (reads_r ? c.r : 0.0);
  };
  const int64_t full = tiles / kPlanCUs, rem = tiles % kPlanCUs;
  return (double)full * round(kPlanCUs) + (rem ? round(rem) : 0.0);
}

// ... of an M x N region
double region_cost(int tile, const TileKind& k, bool reads_r, int64_t M, int64_t N, int64_t nk) {
  const int64_t bn = k.epi == 1 ? kGemmTileDim[tile].n / 2 : kGemmTileDim[tile].n;
  return tiles_cost(tile, k, reads_r, ceil_div(M, kGemmTileDim[tile].m) * ceil_div(N, bn), nk);
}

}  // namespace

// The launch with the least estimated time among
//   * one launch of one tile size;
//   * r whole rounds of 256x256 tiles (one tile per CU and round), the
//     remaining columns or rows as tiles of any size -- a last round that a
//     large tile would leave half empty;
//   * the split-K plan, given a workspace: whole rounds, then the remaining
//     tiles with K split; it pays where few tiles face a long K.
// Larger tiles cost less per FLOP (the 256x256 tile's slice with every CU
// busy: 1.58 us, four 128x128 slices: 2.4 us), smaller ones fill the CUs and
// their last round.
GemmPlan gemm_plan(int transA, int64_t M, int64_t N, int64_t K, int epi, bool reads_r, bool split_k,
                   bool split_rows) {
  const TileKind kind{transA != 0, split_rows, epi};
  const int64_t nk = ceil_div(K, 64);
  GemmPlan best{true, 0, kTile256, kTile256, 1};
  double best_us = 1e30;
  auto offer = [&](const GemmPlan& p, double us) {
    if (us < best_us) {
      best = p;
      best_us = us;
    }
  };
  for (int t = 0; t < kNumGemmTiles; ++t)
    offer(GemmPlan{true, 0, t, t, 1}, region_cost(t, kind, reads_r, M, N, nk));
  const int64_t un = epi == 1 ? 128 : 256;         // output columns per 256-wide tile
  const int64_t tm = ceil_div(M, 256), tc = ceil_div(N, un);
  for (int cols = 0; cols < 2; ++cols) {
    const int64_t across = cols ? tm : tc;         // tiles per tile column (row)
    const int64_t along = cols ? tc : tm;
    const int64_t rounds = tm * tc / kPlanCUs;
    if (rounds < 1 || across > kPlanCUs) continue;
    const int64_t n = rounds * kPlanCUs / across;  // tile columns (rows) in whole rounds
    if (n < 1 || n >= along) continue;
    const double head = tiles_cost(kTile256, kind, reads_r, n * across, nk);
    const int64_t at = n * (cols ? un : 256);
    for (int t = 0; t < kNumGemmTiles; ++t)
      offer(GemmPlan{cols == 1, at, kTile256, t, 1},
            head + kLaunchUs + region_cost(t, kind, reads_r, cols ? M : M - at, cols ? N - at : N, nk));
  }
  SplitTail st;
  if (split_k && epi == 0 && gemm_splitk_tail(M, N, K, &st)) {
    const int64_t tail = ceil_div(st.Mt, 256) * ceil_div(st.Nt, 256);
    const int64_t rest = tm * tc - tail;
    const double sum = 2.0 * 4.0 * st.S * (double)st.Mt * (double)st.Nt / kPartialBytesPerUs;
    offer(GemmPlan{st.columns, st.split_at, kTile256, kTile256, st.S},
          tiles_cost(kTile256, kind, reads_r, rest, nk) + (rest ? kLaunchUs : 0.0) +
              tiles_cost(kTile256, kind, false, tail * st.S, ceil_div(nk, st.S)) + kLaunchUs + sum);
  }
  return best;
}

}  // namespace lt
