// The context layer's host rules and its attention's work list, for the tests:
// reads one case per line from stdin, writes one line of numbers per case.
//   plan H nh nkv ffn batch B C_max
//     -> slots, default W ns parts, parts the static scratch holds, W ns parts there,
//        parts of a workspace created for exactly this call
//   walk nkv B Cmax W ns batch ctx...
//     -> 1 if the workgroups' parts cover every sub-chunk once, in order, at
//        partial numbers of their own below the plan's bound, where the combine
//        looks for them; else 0
//   gemm n0 n1 N K M floats
//     -> tile size and k parts of a projection, the stages of k and the first of
//        each part, and at the end their number
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "xp_layer_plan.h"

using namespace xp;

struct Part {
  long partial;
  int lo, hi;
};

// k_attn's walk of workgroup w (sub-chunks only) and k_attn_comb's search.
static bool walk(int nkv, int W, int ns, const std::vector<int>& subs) {
  const int batch = (int)subs.size();
  std::vector<int> pre(batch + 1, 0);
  for (int b = 0; b < batch; ++b) pre[b + 1] = pre[b] + subs[b];
  const long segs = (long)batch * nkv, bound = ns > 0 ? W : W + segs - 1;
  std::vector<std::vector<Part>> of(segs);
  for (int w = 0; w < W; ++w) {
    if (ns > 0) {
      const int seg = w / ns, i = w % ns, nb = subs[seg / nkv];
      const AttnSegment p(nb, ns);
      if (i < p.n) of[seg].push_back({(long)w, p.first(i), p.first(i + 1)});
      continue;
    }
    const AttnShare share(pre[batch], nkv, W);
    if (w >= share.W) continue;
    long f = share.first(w);
    const long f1 = share.first(w + 1);
    while (f < f1) {
      int b = 0;
      while (b + 1 < batch && (long)pre[b + 1] * nkv <= f) ++b;
      const long in = f - (long)pre[b] * nkv;
      const int kvh = (int)(in / subs[b]), jc = (int)(in % subs[b]);
      const long seg = (long)b * nkv + kvh;
      const int n = (int)std::min<long>(subs[b] - jc, f1 - f);
      of[seg].push_back({w + seg, jc, jc + n});
      f += n;
    }
  }
  std::vector<bool> used(bound, false);
  for (long seg = 0; seg < segs; ++seg) {
    const int b = (int)(seg / nkv), kvh = (int)(seg % nkv), nb = subs[b];
    long pa;
    int n;
    if (ns > 0) {
      pa = seg * ns;
      n = AttnSegment(nb, ns).n;
    } else {
      const AttnShare share(pre[batch], nkv, W);
      const long fa = (long)pre[b] * nkv + (long)kvh * nb;
      const int wa = share.of(fa);
      n = share.of(fa + nb - 1) - wa + 1;
      pa = wa + seg;
    }
    if (n != (int)of[seg].size()) return false;
    int at = 0;
    for (int i = 0; i < n; ++i) {
      const Part& p = of[seg][i];
      if (p.partial != pa + i || p.partial >= bound || used[p.partial]) return false;
      if (p.lo != at || p.hi <= p.lo) return false;
      used[p.partial] = true;
      at = p.hi;
    }
    if (at != nb) return false;
  }
  return true;
}

int main() {
  std::string line, what;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    in >> what;
    if (what == "plan") {
      LayerDims L;
      int batch, B, C;
      in >> L.H >> L.nh >> L.nkv >> L.ffn >> batch >> B >> C;
      L.grp = L.nh / L.nkv;
      const AttnPlan d = attn_plan_default(L, batch, B, C);
      const size_t room = scratch_parts(L, (size_t)batch * B);
      const AttnPlan f = attn_plan_fit(L, batch, B, C, room);
      printf("%zu %d %d %zu %zu %d %d %zu %zu\n", attn_slots(L, B), d.W, d.ns, d.parts, room, f.W,
             f.ns, f.parts, attn_parts_max(L, batch, B));
    } else if (what == "gemm") {
      int n0, n1, N, K, M;
      size_t floats;
      in >> n0 >> n1 >> N >> K >> M >> floats;
      const LayerPlan g = layer_plan(n0, n1, N, K, M, false, floats);
      const int nk = K / gemm_stage_k(g.bn);
      printf("%d %d %d", g.bn, g.S, nk);
      for (int s = 0; s <= g.S; ++s) printf(" %d", SplitParts(nk, g.S).first(s));
      printf("\n");
    } else {
      int nkv, B, Cmax, W, ns, batch;
      in >> nkv >> B >> Cmax >> W >> ns >> batch;
      std::vector<int> subs(batch);
      for (int b = 0; b < batch; ++b) {
        int c;
        in >> c;
        subs[b] = (c + B + kSub - 1) / kSub;
      }
      printf("%d\n", walk(nkv, W, ns, subs) ? 1 : 0);
    }
  }
}
