"""The setup's device-memory arena (csrc/arena.hpp) run over host memory (CPU
only): buffers in use never overlap, memory given back is used again, slabs
that hold nothing are freed."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_09001_amd", "csrc")

HEAD = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include "arena.hpp"
// 4 GiB of addresses, nothing behind them: the arena touches none of the memory it hands out
struct Host {
  static inline std::map<char*, size_t> live;
  static inline size_t held = 0, limit = ~(size_t)0, base = (size_t)1 << 40;
  static char* take(size_t b, bool must) {
    if (held + b > limit) {
      if (must) throw 1;
      return nullptr;
    }
    char* p = (char*)base;
    base += b + 4096;
    live[p] = b;
    held += b;
    return p;
  }
  static void give(char* p) { held -= live.at(p); live.erase(p); }
};
using A = amg::ArenaOf<Host>;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
int main() {
"""


def _run(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(HEAD + body + "\nreturn 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_random_use_does_not_overlap(tmp_path):
    _run(tmp_path, r"""
  std::mt19937 g(7);
  A a;
  std::map<char*, size_t> use;
  for (int i = 0; i < 20000; ++i) {
    if (use.empty() || g() % 5 < 3) {
      const size_t b = 1 + (g() % 3 == 0 ? g() % (1 << 22) : g() % 5000);
      char* p = (char*)a.get(b);
      CHECK(((size_t)p & 255) == 0);
      auto it = use.lower_bound(p);
      CHECK(it == use.end() || p + b <= it->first);
      CHECK(it == use.begin() || std::prev(it)->first + std::prev(it)->second <= p);
      auto s = std::prev(Host::live.upper_bound(p));
      CHECK(p + b <= s->first + s->second);
      use[p] = b;
    } else {
      auto it = use.begin();
      std::advance(it, g() % use.size());
      a.put(it->first, it->second);
      use.erase(it);
    }
  }
  for (auto& u : use) a.put(u.first, u.second);
  a.trim();
  CHECK(a.held() == 0 && Host::live.empty());
""")


def test_memory_given_back_is_used_again(tmp_path):
    _run(tmp_path, r"""
  {
    A a;
    void* p = a.get(1000);
    void* q = a.get(5000);
    void* r = a.get(300);
    a.put(q, 5000);                       // a hole below r
    CHECK(a.get(4096) == q);
    CHECK((char*)a.get(1024) == (char*)q + 4096);
    a.put(r, 300);                        // the end
    CHECK(a.get(512) == r);
    CHECK(Host::live.size() == 1);
    void* big = a.get((size_t)300 << 20); // a slab of its own
    CHECK(Host::live.size() == 2);
    a.put(big, (size_t)300 << 20);
    a.trim();
    CHECK(Host::live.size() == 1 && a.held() == (size_t)2 << 20);
    CHECK(a.get(1000) != p);
    a.reset();
    CHECK(a.get(1000) == p);
  }
  CHECK(Host::live.empty());
""")


def test_a_slab_that_cannot_be_had_leaves_the_request(tmp_path):
    _run(tmp_path, r"""
  Host::limit = (size_t)100 << 20;
  {
    A a;
    CHECK(a.get((size_t)60 << 20));
    CHECK(a.get((size_t)10 << 20));       // a slab would be 60 MB: the request itself
    CHECK(a.held() == (size_t)70 << 20);
    CHECK(a.get((size_t)30 << 20));
    bool thrown = false;
    try { a.get(256); } catch (int) { thrown = true; }
    CHECK(thrown && a.held() == (size_t)100 << 20);
  }
  CHECK(Host::live.empty());
""")


def test_expected_sizes_take_one_slab(tmp_path):
    _run(tmp_path, r"""
  {
    A a;
    a.expect((size_t)40 << 20);
    for (int i = 0; i < 40; ++i) a.get((size_t)1 << 20);
    CHECK(Host::live.size() == 1 && a.held() == (size_t)40 << 20);
    a.get(1000);                          // beyond: a quarter of what is held
    CHECK(Host::live.size() == 2 && a.held() == (size_t)50 << 20);
  }
  {
    A b;
    b.expect((size_t)600 << 20);          // in slabs of at most 256 MB
    for (int i = 0; i < 58; ++i) b.get((size_t)10 << 20);
    CHECK(Host::live.size() == 3 && b.held() == (size_t)600 << 20);
  }
  {
    A c;
    c.expect(1000);                       // at least 2 MB
    c.get(100);
    CHECK(c.held() == (size_t)2 << 20);
  }
  CHECK(Host::live.empty());
""")
