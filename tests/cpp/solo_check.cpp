// Host-only check of the streamed register-owner schedule with solo slots: register
// vertices that have an edge in a class without register slots, whose edge there runs
// as one more slot in the place of the class's last pair slot (reg_schedule.cpp).
// Input on stdin: "n m C" then m lines "u v J colour"; arguments: W nth.
// Decodes rs_words, rs_pwords and rs_act as the kernel reads them (sweep_rstream.hip)
// and prints "equal=.. bad=.. masks=.. solo=.. free=..": every edge exactly once in its
// class with its own roles, entries out of place, wrong mask bits (the last pair slot
// and the solo slot at once among them), solo edges, edges in pair slots.
// Exit status 2: the form does not apply.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <tuple>
#include <vector>

#include "internal.hpp"
int cosm::set_error(int st, const std::string &m) { fprintf(stderr, "err %s\n", m.c_str()); return st; }
void cosm::clear_error() {}

int main(int argc, char **argv) {
  if (argc < 3) return 1;
  const int W = atoi(argv[1]), request = atoi(argv[2]);
  int n; long m; int C;
  if (scanf("%d %ld %d", &n, &m, &C) != 3) return 1;
  cosm_state s; s.n = n; s.m = m; s.C = C;
  std::multiset<std::tuple<int, int, int, int>> want, got;
  for (long k = 0; k < m; k++) {
    int u, v, J, c;
    if (scanf("%d %d %d %d", &u, &v, &J, &c) != 4) return 1;
    s.h_eu.push_back(u); s.h_ev.push_back(v); s.h_J.push_back(J); s.h_colour.push_back(c);
    want.insert({c, u, v, J});
  }
  cosm::LdsSchedule L;
  if (cosm::build_rstream_schedule(s, W, request, &L, true)) {
    puts("ERANGE");
    return 2;
  }
  const int K = L.reg_k, nth = L.nth, nr = L.n_rows, P = cosm::kRStreamPairs, nw = nth / 64;
  const uint32_t rowb = 4u * W;
  long bad = 0, masks = 0, solo = 0, pairs = 0;
  auto dummy = [&](uint32_t row) {
    if (row < (uint32_t)nr || row >= (uint32_t)(nr + cosm::kRStreamDummyRows(W))) bad++;
  };
  // a lane's edge between register row k and an LDS row
  auto owner = [&](int c, int k, int t, uint32_t x, uint32_t y) {
    float J;
    memcpy(&J, &y, 4);
    const uint32_t row = (x & 0x7fffffffu) / rowb;
    if (J == 0.0f) { dummy(row); return false; }
    if (row >= (uint32_t)nr) { bad++; return false; }
    const int v = L.reg_vertex[(size_t)k * nth + t], w = L.slot_vertex[row];
    if (v < 0 || w < 0) { bad++; return false; }
    const bool flip = x >> 31;
    got.insert({c, flip ? w : v, flip ? v : w, (int)J});
    return true;
  };
  size_t j = 0;
  for (int c = 0; c < C; c++) {
    const uint32_t *act = &L.rs_act[(size_t)c * nw];
    bool solo_class = false;
    for (int w = 0; w < nw; w++) {
      if ((act[w] & 1u) != (act[0] & 1u)) masks++;
      solo_class |= (act[w] >> (1 + P)) & 1u;
    }
    if (act[0] & 1u) {
      for (int k = 0; k < K; k++)
        for (int t = 0; t < nth; t++) {
          const size_t i = (j * K + k) * nth + t;
          owner(c, k, t, L.rs_words[2 * i], L.rs_words[2 * i + 1]);
        }
      j++;
    }
    for (int p = 0; p < P; p++)
      for (int t = 0; t < nth; t++) {
        const size_t i = ((size_t)c * P + p) * nth + t;
        const uint32_t x = L.rs_pwords[2 * i], y = L.rs_pwords[2 * i + 1], a = act[t / 64];
        if (p == P - 1 && solo_class) {
          if ((a >> (1 + p)) & 1u) masks++;  // the wave would take the words for a pair's
          if (owner(c, K - 1, t, x, y)) {
            solo++;
            if (!((a >> (1 + P)) & 1u)) masks++;
          }
          continue;
        }
        const int J = (int32_t)x >> 18;
        const uint32_t ru = (x & 0x3ffffu) / rowb, rv = y / rowb;
        if (J == 0) { dummy(ru); dummy(rv); continue; }
        if (!((a >> (1 + p)) & 1u)) masks++;
        if (ru >= (uint32_t)nr || rv >= (uint32_t)nr || L.slot_vertex[ru] < 0 || L.slot_vertex[rv] < 0) {
          bad++;
          continue;
        }
        got.insert({c, L.slot_vertex[ru], L.slot_vertex[rv], J});
        pairs++;
      }
  }
  printf("equal=%d bad=%ld masks=%ld solo=%ld free=%ld\n", (int)(want == got), bad, masks, solo, pairs);
  return 0;
}
