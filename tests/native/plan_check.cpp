// Host check of the grouped weight-gradient plans: for every width, depth and
// token count below, the launch that grouped_weight_grads would make writes
// its bias rows and contraction slices inside the workspace areas laid out for
// them, and the reduction after it reads exactly what was written; its tile is
// one that the launch takes, and a split tail is the launch's last tiles. The
// launches are replaced by recorders; no GPU is touched and no pointer is
// followed.
#include "../../paper_2609_28568_amd/csrc/gpt2.cpp"

#include <cstdio>

static GemmGroupedArgs g_launch;
static ReduceSegs g_reduce;

hipError_t launch_gemm_grouped(const GemmGroupedArgs& g, hipStream_t) {
  g_launch = g;
  return hipSuccess;
}
hipError_t launch_reduce_segs(const ReduceSegs& r, int, hipStream_t) {
  g_reduce = r;
  return hipSuccess;
}

static const ReduceSeg* seg_of(const float* src) {
  for (int i = 0; i < g_reduce.count; ++i)
    if (g_reduce.s[i].src == src) return &g_reduce.s[i];
  return nullptr;
}

int main() {
  int checked = 0, bad = 0;
  for (int C = 64; C <= 2048; C += 64)
    for (int F : {64, C, 2 * C, C * 8 / 3 / 64 * 64 + 64, 3 * C, 4 * C - 64, 4 * C, 4 * C + 64, 5376})
      for (int L : {1, 2, 4, 7, 12})
        for (int T : {1, 65, 130, 999, 2048, 4096, 16384}) {
          gpt2_config c{};
          c.n_layer = L; c.n_head = C / 64; c.d_model = C; c.d_ff = F; c.vocab = 64; c.vocab_padded = 64;
          c.max_seq_len = T; c.B = 1; c.T = T; c.grad_accum = 1;
          gpt2_model m;
          m.cfg = c;
          m.d = dims_of(c);
          m.act = act_layout(m.d);
          m.ws = ws_layout(m.d);
          kind_sizes(m.d, m.kn);
          size_t o = 0;
          for (int k = 0; k < K_NKIND; ++k) m.koff[k] = o, o += m.kn[k];
          auto at = [](size_t a) { return reinterpret_cast<void*>(a); };
          m.buf = {at(1ull << 44), at(2ull << 44), at(3ull << 44), at(4ull << 44),
                   at(5ull << 44), at(6ull << 44), at(7ull << 44)};
          m.stream = nullptr;
          const WsLayout& w = m.ws;
          const size_t ends[] = {w.lnpart, w.gbs_fc, w.gbs_fp, w.ce_stats};   // of splitk, gbs_qkv, gbs_fc, gbs_fp
          const size_t begins[] = {w.splitk, w.gbs_qkv, w.gbs_fc, w.gbs_fp};
          auto fits = [&](const float* p, size_t floats) {
            const size_t a = (size_t)p - (7ull << 44), b = a + 4 * floats;
            for (int i = 0; i < 4; ++i)
              if (a >= begins[i] && b <= ends[i]) return true;
            return false;
          };
          // the training backward, and one block in isolation
          for (int isolated = 0; isolated < 2; ++isolated) {
            const bf16_t* dy = isolated ? static_cast<const bf16_t*>(at(8ull << 44)) : nullptr;
            if (grouped_weight_grads(&m, isolated ? L - 1 : 0, isolated ? 1 : L, 0, dy) != GPT2_OK) return 2;
            long tiles = 0, last = 0;
            for (int i = 0; i < g_launch.ngroups; ++i) {
              const GemmGroup& gr = g_launch.grp[i];
              const int bm = g_launch.bm, bn = g_launch.bn;
              last = (long)((gr.M + bm - 1) / bm) * ((gr.N + bn - 1) / bn) * gr.count * std::max(gr.splits, 1);
              tiles += last;
              if (bm == 192 ? bn != 192 || gr.M % 192 || gr.N % 192 : bn != 128 || (bm != 128 && bm != 256)) return 3;
            }
            if (g_launch.nfull && (g_launch.nfull != tiles - last || g_launch.nfull % 8 || last % 8)) return 4;
            for (int i = 0; i < g_launch.ngroups; ++i) {
              const GemmGroup& gr = g_launch.grp[i];
              const int chunks = gr.splits > 1 ? gr.splits : 1;
              const char* what = nullptr;
              if (gr.bsum) {
                const int rows = chunks * gemm_grouped_bias_parts(g_launch, i);
                const ReduceSeg* s = seg_of(gr.bsum);
                if (!fits(gr.bsum, (size_t)rows * gr.count * gr.M)) what = "bias rows outside their area";
                else if (!s || s->slices != rows || s->stride != (long)gr.count * gr.M)
                  what = "bias rows not all summed";
              }
              if (!what && chunks > 1) {
                const ReduceSeg* s = seg_of(static_cast<const float*>(gr.C));
                if (!fits(static_cast<const float*>(gr.C), (size_t)chunks * gr.split_stride))
                  what = "slices outside their area";
                else if (!s || s->slices != chunks || s->stride != gr.split_stride) what = "slices not all summed";
              }
              ++checked;
              if (what && ++bad <= 10)
                std::printf("C %d F %d L %d T %d %s group %d: %s\n", C, F, L, T, isolated ? "isolated" : "training", i,
                            what);
            }
          }
        }
  std::printf("%d groups checked, %d bad\n", checked, bad);
  return bad ? 1 : 0;
}
