// Host check: what rotconv_pool_fwd_static accepts for average-pooling plans covers what the call goes on to touch.
// The entry points' own source is compiled in, so that its file-local rules are the ones that are checked; everything else comes
// from the built library.  Touches no GPU.  Prints a line for each plan whose accepted need is too small, then their number.
#include "rotconv_api.hip"

#include <cstdio>
#include <cstdlib>
#include <random>

namespace {

// Bytes that rotconv_fwd on this plan writes and reads of its scratch, by the route that f32_rotconv_fwd takes for aligned tensors.
size_t touched(const rotconv_plan* p, const char* ws) {
  if (p->pad_child && p->pad_use[0]) return pad_layout(p).child + touched(p->pad_child, ws);
  if (p->ig[0].mt) return ig_part_bytes(p, p->ig[0]) + ig_fwd_block_bytes(p, p->ig[0]);
  return f32_fwd_need(p, ws, ws, ws);
}

}  // namespace

int main(int argc, char** argv) {
  std::mt19937 gen(argc > 1 ? std::atoi(argv[1]) : 1);
  auto pick = [&](int lo, int hi) { return (int)(lo + gen() % (unsigned)(hi - lo + 1)); };
  int plans = 0, bad = 0, routed = 0;
  while (plans < 4000) {
    rotconv_desc d{};
    d.N = pick(1, 4); d.Cin = pick(1, 4); d.Cout = pick(8, 80); d.R = pick(0, 1) ? 4 : 1;
    d.H = pick(30, 1400); d.W = pick(15, 700) | 1;
    const double staged = 4.0 * d.N * (d.Cin + d.Cout) * d.H * d.W;
    if (staged > 18e6 || staged < 2e6) continue;
    d.k = 3; d.stride = 1; d.pad = 1; d.pool_op = ROTCONV_POOL_AVG; d.mode = ROTCONV_EXACT90;
    d.dtype = pick(0, 3) ? ROTCONV_F32 : ROTCONV_BF16;
    rotconv_plan* p = nullptr;
    if (rotconv_plan_create(&d, &p) != ROTCONV_OK) continue;
    ++plans;
    const char* at = reinterpret_cast<const char*>((uintptr_t)1 << 40);       // aligned; nothing is read
    const size_t need = pool_fwd_need(p, at, at, at, nullptr, at);
    const size_t front = d.dtype == ROTCONV_BF16 ? p->ws_bytes - p->ws_inner : 0;
    const size_t real = front + avg_layout(p).child + touched(p->avg_child, at);
    if (need <= kStaticScratchBytes) {
      ++routed;
      if (real > need || real > kStaticScratchBytes) {
        if (++bad <= 5)
          std::printf("N=%d %d -> %d, %dx%d R=%d dtype=%d: accepted with %zu bytes, touches %zu\n", d.N, d.Cin, d.Cout, d.H, d.W, d.R,
                      d.dtype, need, real);
      }
    }
    rotconv_plan_destroy(p);
  }
  std::printf("plans %d accepted %d too small %d\n", plans, routed, bad);
  return bad ? 1 : 0;
}
