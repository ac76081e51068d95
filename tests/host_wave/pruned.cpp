// Test infrastructure: the pruned layer step (csrc/gbmw_pruned.h) on the CPU, one problem per run.
//   pruned <in> <out>
// in:  int32 S, E, L, unit, records | c [L][S] f32 | M [L][S] i32 | R [L][S][S] f32
// out: C [L][E+1][S] f32 as the readers of the tables see it | records [L][E+1][S] bytes (layers >= 1)
// Every buffer has exactly the size that the library gives it, cells, records and LDS start as
// values that no result contains, so that a read of one that was never written shows in the output.
#include <vector>

#include <hip/hip_runtime.h>

namespace {

// in here, so that the LDS variables of its templates are this file's own: the sanitizer guards no others
#include "gbmw_pruned.h"

using namespace gbmw;

template <typename T>
std::vector<T> read_n(FILE* f, size_t n) {
  std::vector<T> v(n);
  if (fread(v.data(), sizeof(T), n, f) != n) { fprintf(stderr, "short input\n"); exit(2); }
  return v;
}

template <int NCH, int KEEP, bool FIRST, bool ARG>
void layer(const Tables& t, int l, int unit) {
  const int groups = (t.E + 64) / 64;                    // as pruned_shape
  const int places = unit == 0 ? groups : (groups + kWaves * unit - 1) / (kWaves * unit);
  const size_t words = (size_t)pruned_lds_floats(t.S, KEEP);
  for (int place = 0; place < places; ++place) {
    std::vector<uint32_t> lds(words, 0x7fdeadadu);       // a fresh allocation of this size for every workgroup
    host_wave::run([&] {
      pruned_step<NCH, KEEP, FIRST, ARG, false>(t, l, t.perm[0], place, places, unit, reinterpret_cast<float*>(lds.data()));
    });
  }
}

template <int NCH, int KEEP>
void layer(const Tables& t, int l, int unit) {
  if (t.A) { if (l == 1) layer<NCH, KEEP, true, true>(t, l, unit); else layer<NCH, KEEP, false, true>(t, l, unit); }
  else { if (l == 1) layer<NCH, KEEP, true, false>(t, l, unit); else layer<NCH, KEEP, false, false>(t, l, unit); }
}

void layer(const Tables& t, int l, int unit) {
  if (t.S > 128) layer<4, kept(256)>(t, l, unit);
  else if (t.S > 64) layer<2, kept(128)>(t, l, unit);
  else if (t.SP == 4) layer<1, kept(4)>(t, l, unit);
  else if (t.SP == 8) layer<1, kept(8)>(t, l, unit);
  else if (t.SP == 12) layer<1, kept(12)>(t, l, unit);
  else layer<1, kept(16)>(t, l, unit);
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  FILE* f = fopen(argv[1], "rb");
  if (!f) return 2;
  const std::vector<int> h = read_n<int>(f, 5);
  const int S = h[0], E = h[1], L = h[2], unit = h[3], records = h[4];
  const int EP = (E + 1 + 255) / 256 * 256, G = EP / 64;
  const std::vector<float> c = read_n<float>(f, (size_t)L * S);
  const std::vector<int> M = read_n<int>(f, (size_t)L * S);
  const std::vector<float> R = read_n<float>(f, (size_t)L * S * S);
  fclose(f);

  std::vector<uint32_t> C((size_t)L * S * EP, 0x7fbadbadu);
  std::vector<float> Rn((size_t)L * S * S);
  std::vector<float4> Row((size_t)L * S);
  std::vector<float2> sums((size_t)L * S * G, float2{-1.0f, -2.0f});
  std::vector<uint8_t> A(records ? (size_t)L * S * EP : 0, 0xEE), Asum(records ? (size_t)L * S * G : 0, 0xEE);
  const std::vector<int> Ls{L}, off{0};
  const std::vector<int2> perm{{0, 0}};
  Tables t{};
  t.B = 1; t.S = S; t.SP = (S + 3) / 4 * 4; t.E = E; t.EP = EP; t.keep_all = 1; t.runs = 1;
  t.L = Ls.data(); t.off = off.data(); t.perm = perm.data();
  t.c = c.data(); t.M = M.data(); t.Rn = Rn.data(); t.Row = Row.data();
  t.Cbuf = reinterpret_cast<float*>(C.data()); t.Tsum = sums.data();
  t.A = records ? A.data() : nullptr; t.Asum = records ? Asum.data() : nullptr;

  for (int l = 1; l < L; ++l)
    for (int s0 = 0; s0 < S; s0 += 16)
      host_wave::run([&] {                               // as k_prepare_runs: one wave per four rows
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, s = s0 + 4 * wave;
        if (s < S)
          row_limits<4>(R.data() + (size_t)l * S * S, S, s, lane, c.data() + (size_t)l * S, M.data() + (size_t)l * S,
                        Rn.data() + (size_t)l * S * S, Row.data() + (size_t)l * S);
      });
  for (int s = 0; s < S; ++s) {                          // as k_init_layer0
    float* cells = t.Cbuf + (size_t)s * EP;
    for (int e = 0; e < EP; ++e) cells[e] = (M[s] >= 0 && e >= M[s] && e <= E) ? c[s] : INFINITY;
    for (int g = 0; g <= E / 64; ++g) sums[(size_t)s * G + g] = make_float2(c[s], c[s]);
  }
  for (int l = 1; l < L; ++l) layer(t, l, unit);

  f = fopen(argv[2], "wb");
  if (!f) return 2;
  for (int l = 0; l < L; ++l)
    for (int e = 0; e <= E; ++e)
      for (int s = 0; s < S; ++s) {
        const float v = table_cell(t, t.Cbuf + (size_t)l * S * EP, t.Tsum + (size_t)l * S * G, t.M + (size_t)l * S, s, e);
        fwrite(&v, 4, 1, f);
      }
  for (int l = 0; l < L; ++l)
    for (int e = 0; e <= E; ++e)
      for (int s = 0; s < S; ++s) {
        const uint8_t a = (uint8_t)(l == 0 ? 0 : pred_strategy(t, l, s, e));
        fwrite(&a, 1, 1, f);
      }
  fclose(f);
  return 0;
}
