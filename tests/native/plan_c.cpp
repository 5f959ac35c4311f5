// The library's own plans (csrc/linear_plan.h, csrc/attn_plan.h) behind C
// functions, for the index tests.
#include "attn_plan.h"
#include "linear_plan.h"

using namespace smem;

namespace {
template <class C>
void cfg(int* o) {
  const int v[] = {C::BM, C::BN, C::BK, C::NS, C::NW, C::WM, C::WN, C::IA, C::IB, C::RPI, C::CPR, C::STAGE, C::PER_CU};
  for (int i = 0; i < 13; ++i) o[i] = v[i];
}

// F applied to the tile of a head width
template <class F>
int of_width(int dh, F f) {
  return dh == 32 ? f(PageRing<32>()) : dh == 64 ? f(PageRing<64>()) : f(PageRing<128>());
}
template <class P>
void par(int* o) {
  const int v[] = {P::G, P::NSP, P::IPW, P::THREADS, P::ROWS, P::RING, P::OFF_IN, P::OFF_NULL, P::BYTES, P::STATE};
  for (int i = 0; i < 10; ++i) o[i] = v[i];
}
}  // namespace

extern "C" {
int lp_lin_chunk(int K) { return lin_chunk(K); }
int lp_xcd_grid(int T) { return xcd_grid(T); }
int lp_xcd_order(int i, int T) { return xcd_order(i, T); }

int lp_few_put(int r, int s) { return FewTile::put(r, s); }
int lp_few_get(int lane, int t) { return FewTile::get(lane, t); }
int lp_few_kind(int M, int N, int K) { return few_kind(M, N, K); }
void lp_few_plan(int kind, int K, int* o) {    // row tiles, column tiles, waves, loop, LDS bytes
  const FewPlan& p = kFewPlans[kind];
  o[0] = p.rt, o[1] = p.g, o[2] = few_waves(p, K), o[3] = p.loop, o[4] = (int)few_lds_bytes(p, K);
}
int lp_few_ln_kind(int M, int N, int K) { return few_ln_kind(M, N, K); }
void lp_few_ln_plan(int kind, int K, int* o) { // row tiles, column tiles, waves per chunk, steps, threads, LDS bytes
  const FewLnPlan& p = kFewLnPlans[kind];
  o[0] = p.rt, o[1] = p.g, o[2] = p.wpc, o[3] = p.u, o[4] = few_ln_threads(p, K), o[5] = (int)few_ln_lds_bytes(p, K);
}
int lp_wide_fits(int M, int N, int K) { return wide_fits(M, N, K); }
int lp_wide_lds(int rt, int K) { return wide_lds(rt, K); }

int lp_gemm_tile(int M, int N, int K) { return gemm_tile(M, N, K); }
void lp_gemm_cfg(int tile, int* o) {
  switch (tile) {
    case kGemmWide: cfg<GemmWide>(o); break;
    case kGemmTall: cfg<GemmTall>(o); break;
    case kGemmPair: cfg<GemmPair>(o); break;
    case kGemmSmall: cfg<GemmSmall>(o); break;
    default: cfg<GemmBrief>(o); break;
  }
}
int lp_gemm_swz(int tile, int r) {
  switch (tile) {
    case kGemmWide: return GemmWide::swz(r);
    case kGemmTall: return GemmTall::swz(r);
    case kGemmPair: return GemmPair::swz(r);
    case kGemmSmall: return GemmSmall::swz(r);
    default: return GemmBrief::swz(r);
  }
}
int lp_gemm_place(int i, int tiles_m, int tiles_n) {   // row tile * tiles_n + column tile, or -1
  const GemmPlace p = gemm_place(i, tiles_m, tiles_n);
  return p.ok ? p.tm * tiles_n + p.tn : -1;
}
int lp_gemm_grid(int per_cu, int T) { return gemm_grid(per_cu, T); }

int ap_score_key(int kt, int i) { return score_key(kt, i); }
int ap_xcd_range(int n, int all) { return xcd_range(n, all); }
void ap_ring(int dh, int* o) {                 // tile bytes, key plane bytes, key row bytes, stages, instructions per wave
  of_width(dh, [&](auto r) {
    using R = decltype(r);
    const int v[] = {R::TILE, R::KBYTES, R::KRB, R::NS, R::IPW};
    for (int i = 0; i < 5; ++i) o[i] = v[i];
    return 0;
  });
}
int ap_tile_row(int key) { return PageRing<32>::tile_row(key); }
int ap_source(int dh, int byte) { return of_width(dh, [&](auto r) { return decltype(r)::source(byte); }); }
int ap_key_at(int dh, int row, int c) { return of_width(dh, [&](auto r) { return decltype(r)::key_at(row, c); }); }
int ap_value_at(int dh, int d, int key) { return of_width(dh, [&](auto r) { return decltype(r)::value_at(d, key); }); }
int ap_operand_at(int dh, int lane, int dt, int c) {
  return of_width(dh, [&](auto r) { return decltype(r)::operand_at(decltype(r)::operand_lane(lane), dt, c); });
}
int ap_par_row_waves(int n_pairs) { return par_row_waves(n_pairs); }
int ap_par_grid(int n_pairs, int qw) { return par_grid(n_pairs, qw); }
int ap_par_pair(int n, int qw) { return par_pair(n, qw); }
int ap_par_part(int n, int qw) { return par_part(n, qw); }
void ap_par(int dh, int qw, int* o) {          // groups, stages, instructions, threads, rows, LDS offsets, state bytes
  if (dh == 32) qw == 1 ? par<ParLds<32, 1>>(o) : par<ParLds<32, 2>>(o);
  else qw == 1 ? par<ParLds<64, 1>>(o) : par<ParLds<64, 2>>(o);
}
}
