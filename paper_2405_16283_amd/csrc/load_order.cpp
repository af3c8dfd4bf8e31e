// The order in which inputs are loaded where GPU memory does not prescribe one.
//
// The serial order a memgraph is compiled for walks through the program stripe by stripe (or level by level), and loads
// sorted by their first reader follow it: the first rows of x, every weight, and only then the other rows of x, with seven eighths of the
// kernels waiting for them on an idle link (one layer of 64 heads, ffn 22016, 8192 tokens: rows from 1024 on arrive 30 ms
// after the start), or brings all of x, with no weight to multiply it by.  What matters is how early kernels can run.  So loads are
// taken in bundles: of all kernels, the one whose missing inputs unlock the most kernel time per byte, counting every
// kernel that misses the same inputs.  For a product of rows and weights that means both in turn: with a stripes of rows and b
// panels of columns here, the next stripe unlocks b products, the next panel a.  Serial order and this one: 65B-shaped layer 44.5
// and 37.9 ms, fine-tuning step of four sequences of 4096 tokens 33.8 and 30.0, layer on 16384 tokens 16.9 and 15.8.
//
// Kernels that become ready a few at a time are launched in smaller groups, so the serial order stays where the other one is not
// expected to save at least kWorthwhile of the time (scores as tensors, 2048 tokens, where the link has to carry all of
// its 110 MB in either order: 2.66 and 3.04 ms).
#include "load_order.h"

#include <algorithm>
#include <cstring>
#include <unordered_map>

namespace tn {
namespace {

// Sets of loads are bit sets; what all of them may take together, and how many sets the search may look at, about a quarter of a second
constexpr uint64_t kMaxSetBytes = 64ull << 20, kMaxSteps = 50ull << 20;

constexpr double kWorthwhile = 0.04;
constexpr double kLinkBytes = 54e9;  // per second

// (the multipliers are those of splitmix64, whose last steps `mix` is)
uint64_t hash_words(const uint64_t* w, size_t n) {
  uint64_t h = 0x9E3779B97F4A7C15ull;
  for (size_t i = 0; i < n; ++i) {
    h ^= w[i] + 0x9E3779B97F4A7C15ull + (h << 6) + (h >> 2);
    h *= 0xBF58476D1CE4E5B9ull;
    h ^= h >> 29;
  }
  return h;
}

uint64_t mix(uint64_t z) {
  z *= 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

}  // namespace

void order_loads(const MemGraph& mg, const std::vector<double>& seconds, std::vector<int64_t>& key) {
  const int64_t nv = (int64_t)mg.v.size();
  // loads, and how much of them waits for nothing
  std::vector<char> waits(nv, 0);
  for (const auto& e : mg.edges) waits[e.to] = 1;
  std::vector<int64_t> loads;
  std::vector<int32_t> bit(nv, -1);
  uint64_t free_bytes = 0, all_bytes = 0;
  int64_t n_ops = 0;
  for (int64_t m = 0; m < nv; ++m) {
    n_ops += mg.v[m].kind == TN_MG_OP;
    if (mg.v[m].kind != TN_MG_LOAD) continue;
    all_bytes += mg.v[m].bytes;
    if (!waits[m]) free_bytes += mg.v[m].bytes;
    loads.push_back(m);
  }
  // Where more than a tenth has to wait for memory, the places that loads wait for become free in the serial order.  The few that wait in
  // other programs take their turn as soon as they may.
  if (loads.size() < 2 || free_bytes < all_bytes - all_bytes / 10) return;
  const size_t words = (loads.size() + 63) / 64;
  if ((uint64_t)n_ops * words * 8 > kMaxSetBytes) return;
  std::sort(loads.begin(), loads.end(), [&](int64_t a, int64_t b) { return key[a] < key[b]; });
  for (size_t k = 0; k < loads.size(); ++k) bit[loads[k]] = (int32_t)k;

  // the loads every kernel needs, directly or through what it reads, in a topological order
  std::vector<int64_t> by_pos(nv);
  for (int64_t m = 0; m < nv; ++m) by_pos[m] = m;
  std::sort(by_pos.begin(), by_pos.end(), [&](int64_t a, int64_t b) { return mg.v[a].order_pos < mg.v[b].order_pos; });
  std::vector<int64_t> row(nv, -1);
  std::vector<uint64_t> sets;
  sets.reserve((size_t)n_ops * words);
  std::vector<uint64_t> cur(words);
  struct Class { size_t set; double gain; };  // kernels that need the same loads
  std::vector<Class> classes;
  std::unordered_map<uint64_t, std::vector<size_t>> found;
  for (int64_t m : by_pos) {
    const MVertex& x = mg.v[m];
    if (x.kind == TN_MG_INPUT || x.kind == TN_MG_LOAD || x.kind == TN_MG_DROP) continue;
    std::fill(cur.begin(), cur.end(), 0);
    for (int64_t o : x.operands) {
      if (bit[o] >= 0) cur[bit[o] >> 6] |= 1ull << (bit[o] & 63);
      if (row[o] >= 0)
        for (size_t i = 0; i < words; ++i) cur[i] |= sets[(size_t)row[o] * words + i];
    }
    const uint64_t h = hash_words(cur.data(), words);
    auto& list = found[h];
    size_t c = classes.size();
    for (size_t k : list)
      if (!memcmp(&sets[classes[k].set * words], cur.data(), words * 8)) c = k;
    if (c == classes.size()) {
      list.push_back(c);
      classes.push_back({sets.size() / words, 0.0});
      sets.insert(sets.end(), cur.begin(), cur.end());
    }
    row[m] = (int64_t)classes[c].set;
    if (x.kind == TN_MG_OP) classes[c].gain += seconds[m];
  }

  // When all kernels are done if loads arrive in an order: whatever load comes last to a kernel, that kernel and those that come after
  // it are still to be run.
  auto finish = [&](const std::vector<int64_t>& order) {
    std::vector<double> released(order.size(), 0.0);  // kernel time that waits for this load and no later one
    std::vector<size_t> place(order.size());
    for (size_t k = 0; k < order.size(); ++k) place[bit[order[k]]] = k;
    double rest = 0.0, done = 0.0;
    for (const Class& c : classes) {
      const uint64_t* s = &sets[c.set * words];
      size_t last = 0;
      for (size_t i = 0; i < words; ++i)
        for (uint64_t w = s[i]; w; w &= w - 1) last = std::max(last, place[i * 64 + __builtin_ctzll(w)]);
      released[last] += c.gain;
      rest += c.gain;
    }
    double t = 0.0;
    for (size_t k = 0; k < order.size(); ++k) {
      t += mg.v[order[k]].bytes / kLinkBytes;
      done = std::max(done, t + rest);
      rest -= released[k];
    }
    return done;
  };
  const double serial = finish(loads);
  {  // no order is faster than the link or the kernels by themselves
    double link = 0.0, run = 0.0;
    for (int64_t m : loads) link += mg.v[m].bytes / kLinkBytes;
    for (const Class& c : classes) run += c.gain;
    if (std::max(link, run) > (1.0 - kWorthwhile) * serial) return;
  }

  // The search.  A class keeps what it misses as the exclusive or of its loads' numbers and as a sum of bytes, so that taking a load
  // costs a step per class that needs it; a bundle is what the classes with one such number miss.
  std::vector<uint32_t> user_start(loads.size() + 1, 0);
  auto each_load = [&](const Class& c, auto&& f) {
    const uint64_t* s = &sets[c.set * words];
    for (size_t i = 0; i < words; ++i)
      for (uint64_t w = s[i]; w; w &= w - 1) f(i * 64 + (size_t)__builtin_ctzll(w));
  };
  uint64_t n_users = 0;
  for (const Class& c : classes) each_load(c, [&](size_t l) { ++user_start[l + 1]; ++n_users; });
  if (n_users > kMaxSetBytes / 4) return;
  for (size_t l = 0; l < loads.size(); ++l) user_start[l + 1] += user_start[l];
  std::vector<uint32_t> users(n_users), at(user_start.begin(), user_start.end() - 1);
  std::vector<uint64_t> miss(classes.size(), 0), miss_bytes(classes.size(), 0), number(loads.size());
  for (size_t l = 0; l < loads.size(); ++l) number[l] = mix(l + 1);
  std::vector<uint32_t> open;
  for (size_t k = 0; k < classes.size(); ++k) {
    each_load(classes[k], [&](size_t l) {
      users[at[l]++] = (uint32_t)k;
      miss[k] ^= number[l];
      miss_bytes[k] += mg.v[loads[l]].bytes;
    });
    if (miss_bytes[k]) open.push_back((uint32_t)k);
  }
  struct Bundle { uint64_t miss, round; double gain; uint32_t first; };
  size_t slots = 16;
  while (slots < 2 * classes.size()) slots *= 2;
  std::vector<Bundle> table(slots, Bundle{0, 0, 0.0, 0});
  std::vector<uint32_t> touched;
  std::vector<char> taken(loads.size(), 0);
  std::vector<int64_t> picked;
  picked.reserve(loads.size());
  for (uint64_t round = 1, steps = 0; !open.empty() && steps < kMaxSteps; ++round) {
    steps += open.size();
    touched.clear();
    size_t left = 0;
    for (uint32_t k : open) {
      if (!miss_bytes[k]) continue;  // everything it needs is on its way
      open[left++] = k;
      size_t p = miss[k] & (slots - 1);
      while (table[p].round == round && table[p].miss != miss[k]) p = (p + 1) & (slots - 1);
      if (table[p].round != round) {
        table[p] = {miss[k], round, 0.0, k};
        touched.push_back((uint32_t)p);
      }
      table[p].gain += classes[k].gain;
    }
    open.resize(left);
    uint32_t best = 0;
    double best_rate = -1.0;
    for (uint32_t p : touched)  // (of equal ones the one met first: the first in the serial order)
      if (const double rate = table[p].gain / (double)miss_bytes[table[p].first]; rate > best_rate) {
        best_rate = rate;
        best = table[p].first;
      }
    if (best_rate < 0.0) break;
    each_load(classes[best], [&](size_t l) {
      if (taken[l]) return;
      taken[l] = 1;
      picked.push_back(loads[l]);
      for (uint32_t u = user_start[l]; u < user_start[l + 1]; ++u) {
        miss[users[u]] ^= number[l];
        miss_bytes[users[u]] -= mg.v[loads[l]].bytes;
      }
    });
  }
  // loads no kernel needs, and what is left of a search that took too long, in the serial order
  for (size_t k = 0; k < loads.size(); ++k)
    if (!taken[k]) picked.push_back(loads[k]);
  if (finish(picked) > (1.0 - kWorthwhile) * serial) return;
  std::vector<int64_t> keys;
  for (int64_t m : loads) keys.push_back(key[m]);  // ascending
  for (size_t k = 0; k < picked.size(); ++k) key[picked[k]] = keys[k];
}

}  // namespace tn
