// Prints which tile or attention form csrc/plan.h chooses: one answer per line
// of standard input.
//   bf16|fp32 M N K qkv(0|1)            -> tile
//   bounded|running|attn_fp32 T heads   -> form
//   table bf16|fp32|bounded|running     -> every entry
#include <cstdio>
#include <cstring>

#include "plan.h"

using namespace wam;

// rows x columns x waves
void say(const TileCfg& t) { std::printf("%dx%dx%d ", t.bm, t.bn, t.wgm * t.wgn); }
// form : query tiles per wave x waves
void say(const AttnCfg& c) { std::printf("%d:%dx%d ", c.form, c.qt, c.nw); }

template <typename Entry, int N>
void table(const Entry (&t)[N]) {
  for (const Entry& e : t) say(e);
  std::printf("\n");
}

template <int N>
bool gemm(const TileCfg (&t)[N], int m) {
  int n, k, qkv;
  if (std::scanf("%d %d %d", &n, &k, &qkv) != 3) return false;
  const int c = plan_gemm(t, m, n, k, qkv != 0);
  if (c >= 0) say(t[c]);
  std::printf("\n");
  return true;
}

template <int N>
bool attn(const AttnCfg (&t)[N], int T) {
  int heads;
  if (std::scanf("%d", &heads) != 1) return false;
  say(t[plan_attention(t, T, heads)]);
  std::printf("\n");
  return true;
}

int main() {
  char type[16];
  int rows, heads;
  while (std::scanf("%15s", type) == 1) {
    bool ok = true;
    if (!std::strcmp(type, "table")) {
      if (std::scanf("%15s", type) != 1) return 1;
      if (!std::strcmp(type, "bf16")) table(kCfgs);
      else if (!std::strcmp(type, "fp32")) table(kF32Cfgs);
      else if (!std::strcmp(type, "bounded")) table(kBounded);
      else table(kRunning);
      continue;
    }
    if (std::scanf("%d", &rows) != 1) return 1;
    if (!std::strcmp(type, "bf16")) ok = gemm(kCfgs, rows);
    else if (!std::strcmp(type, "fp32")) ok = gemm(kF32Cfgs, rows);
    else if (!std::strcmp(type, "bounded")) ok = attn(kBounded, rows);
    else if (!std::strcmp(type, "running")) ok = attn(kRunning, rows);
    else if ((ok = std::scanf("%d", &heads) == 1)) std::printf("%d\n", plan_attention_f32(rows, heads));
    if (!ok) return 1;
  }
  return 0;
}
