// The library's host-side plans behind a C interface: the tests ask which
// kernels a call runs as.
#include "../paper_2606_10415_amd/csrc/kernels.hpp"

extern "C" {

// out: columns, split_at, head tile (m, n), tail tile (m, n), splits
void query_gemm_plan(int transA, int64_t M, int64_t N, int64_t K, int epi, int reads_r, int split_k, int split_rows,
                     int64_t* out) {
  const lt::GemmPlan p = lt::gemm_plan(transA, M, N, K, epi, reads_r, split_k, split_rows);
  const lt::GemmTileDim h = lt::kGemmTileDim[p.head], t = lt::kGemmTileDim[p.tail];
  const int64_t v[7] = {p.columns, p.split_at, h.m, h.n, t.m, t.n, p.splits};
  for (int i = 0; i < 7; ++i) out[i] = v[i];
}

// key tile width; shares of each key tile into n[] (all 1 when not split)
int query_attn_shares(int B, int S, int Hq, int Hkv, int D, int causal, int* n, int* tiles) {
  const lt::DkdvPlan p = lt::attn_bwd_dkdv_plan(B, S, Hq, Hkv);
  lt::DkdvShares s;
  const bool split = lt::attn_bwd_shares(B, S, Hq, Hkv, D, causal, p, &s);
  *tiles = (S - 1) / p.ktile + 1;
  for (int j = 0; j < *tiles && j < lt::kMaxSplitTiles; ++j) n[j] = split ? s.off[j + 1] - s.off[j] : 1;
  return p.ktile;
}

}  // extern "C"
