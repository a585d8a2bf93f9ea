// Workgroups that hand values to their eight neighbours through mailboxes whose
// stores land late and in any order (only stores of one workgroup to one word
// keep theirs).  Usage: model words|emptied GY GZ LAUNCHES SEED.
//   words    the words of sor_mail.h
//   emptied  the values themselves in four slot sets, emptied by the reader
// Prints "ok", or what went wrong, and exits with 0 / 1.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <random>
#include <vector>

#include "sor_mail.h"

using namespace ek;

constexpr uint64_t EMPTY = 0xFFF7A5C35A3C7F11ull;
static_assert(EMPTY == SOR_UNSENT, "both start with the same word in every slot");

struct Store {
  int writer;
  size_t at;
  uint64_t value;
  bool lazy;           // an emptying store: lands when nothing else can happen
};

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const bool words = !std::strcmp(argv[1], "words");
  const int gy = std::atoi(argv[2]), gz = std::atoi(argv[3]), launches = std::atoi(argv[4]), W = gy * gz;
  std::mt19937_64 rng(std::atoi(argv[5]));
  const int sets = words ? SOR_SETS : 4;
  std::vector<uint64_t> mail((size_t)SOR_BANKS * sets * W * 8, EMPTY);
  int bank = 0;
  auto slot_of = [&](int in_bank, int set, int wg, int dir) {
    return (((size_t)in_bank * sets + set) * W + wg) * 8 + dir;
  };
  const int dy[8] = {-1, 1, 0, 0, -1, 1, -1, 1}, dz[8] = {0, 0, -1, 1, -1, -1, 1, 1};
  const int opposite[8] = {1, 0, 3, 2, 7, 6, 5, 4};
  auto neighbour = [&](int wg, int dir) {
    return (wg / gy + dz[dir] + gz) % gz * gy + (wg % gy + dy[dir] + gy) % gy;
  };
  // what a workgroup sends after an iteration: few values, so that they repeat,
  // the special words among them
  auto sent = [&](int wg, int n, int dir) {
    const uint64_t v[4] = {0, 1, words ? SOR_AGAIN : 2, words ? SOR_UNSENT : 3};
    return v[(wg * 7 + n / 3 + dir * n % 5) % 4];
  };

  int base = 0;
  for (int l = 0; l < launches; ++l) {
    const int n_it = 1 + int(rng() % 12);
    const bool abandoned = words && rng() % 4 == 0;       // a workgroup gives up somewhere
    auto slot = [&](int set, int wg, int dir) { return slot_of(words ? bank : 0, set, wg, dir); };
    std::deque<Store> pending;
    struct Group {
      int it = 0;                // iteration sent last
      bool sending = true, gone = false;
      int next = 0;              // direction of the next store or read
      unsigned have = 0;         // directions received
      uint64_t got[2][8], gave[2][8];
    };
    std::vector<Group> g(W);
    for (auto& w : g) {
      w.it = 1;
      for (int k = 0; k < 16; ++k) w.got[k / 8][k % 8] = w.gave[k / 8][k % 8] = SOR_UNSENT;
    }
    auto post = [&](int writer, size_t at, uint64_t v, bool lazy) { pending.push_back({writer, at, v, lazy}); };
    auto land = [&](size_t k) {
      // the writer's earlier stores to the word land first
      for (size_t j = 0; j < k; ++j)
        if (pending[j].at == pending[k].at && pending[j].writer == pending[k].writer) { k = j; break; }
      mail[pending[k].at] = pending[k].value;
      pending.erase(pending.begin() + k);
    };
    if (words)
      for (int w = 0; w < W; ++w)
        for (int k = 0; k < 8 * sets; ++k) post(w, slot_of(bank ^ 1, k / 8, w, k % 8), SOR_UNSENT, false);
    // one step of a workgroup; false: it polled and found nothing new
    auto advance = [&](int w) -> bool {
      Group& G = g[w];
      const int number = base + G.it, set = words ? G.it & 1 : G.it & 3, dir = G.next;
      G.next = (G.next + 1) % 8;
      if (G.sending) {
        uint64_t v = sent(w, number, dir);
        if (words) {
          v = sor_word(v, G.gave[0][dir]);
          G.gave[0][dir] = G.gave[1][dir];
          G.gave[1][dir] = v;
        }
        post(w, slot(set, neighbour(w, dir), opposite[dir]), v, false);
        if (G.next == 0) { G.sending = false; G.have = 0; }
        return true;
      }
      uint64_t v = mail[slot(set, w, dir)];
      for (const Store& p : pending)   // a workgroup sees its own stores
        if (p.writer == w && p.at == slot(set, w, dir)) v = p.value;
      const bool got = !(G.have >> dir & 1) && v != (words ? G.got[0][dir] : EMPTY);
      if (got) {
        uint64_t want = sent(neighbour(w, dir), number, opposite[dir]), value = v;
        if (words) {
          if (want == SOR_UNSENT || want == SOR_AGAIN) want ^= 4;
          value = sor_value(v, G.got[0][dir]);
          G.got[0][dir] = G.got[1][dir];
          G.got[1][dir] = v;
        }
        if (value != want) {
          std::printf("a wrong value was taken (launch %d)\n", l);
          std::exit(1);
        }
        if (!words) post(w, slot(set, w, dir), EMPTY, true);
        G.have |= 1u << dir;
      }
      if (G.have == 255u) {
        G.next = 0;
        G.sending = true;
        if (G.it == n_it) G.gone = true;
        ++G.it;
      }
      return got;
    };
    if (abandoned) {
      // some steps, then every workgroup ends where it is
      for (int k = int(rng() % 400); k > 0; --k) {
        const int w = int(rng() % W);
        if (!g[w].gone) advance(w);
        if (!pending.empty() && rng() % 3 == 0) land(rng() % pending.size());
      }
    } else {
      long long idle = 0;
      for (;;) {
        bool all = true;
        for (auto& w : g) all = all && w.gone;
        if (all) break;
        const int w = int(rng() % W);
        if (!g[w].gone && advance(w)) idle = 0;
        else ++idle;
        if (!pending.empty() && rng() % 4 == 0) {
          const size_t k = rng() % pending.size();
          if (!pending[k].lazy) { land(k); idle = 0; }
        }
        if (idle > 400ll * W) {          // only the stores held back are left, or none
          if (pending.empty()) {
            std::printf("a value was lost: every workgroup waits (launch %d)\n", l);
            return 1;
          }
          land(rng() % pending.size());
          idle = 0;
        }
      }
    }
    while (!pending.empty()) land(0);    // a launch's stores have landed when it ends
    base += n_it;
    bank ^= 1;
  }
  std::printf("ok\n");
  return 0;
}
