"""The packed request entry of a joined launch (rg_internal.h), compiled for
the host (no GPU): every entry that packs unpacks to the same numbers, and one
past a field's last value is refused."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_34388_amd", "csrc")
ROCM = "/opt/rocm/include"

SOURCE = r"""
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <functional>

#include "rg_internal.h"

using namespace rg;

// Every number of an entry by itself.
struct Fields {
  uint32_t q_start, n, ctx, nv, page_start, item_start, rows[3], prefix[3], lead[3], count, step, last;
};

static AttnReqBr entry(const Fields& f) {
  AttnReqBr r;
  std::memset(&r, 0, sizeof(r));
  r.q_start = (int32_t)f.q_start;
  r.ctx = (int32_t)f.ctx;
  r.nv = (int32_t)(f.n | f.nv << 16);
  r.page_start = (int32_t)f.page_start;
  r.item_start = (int32_t)f.item_start;
  for (int b = 0; b < 3; ++b) r.br[b] = (int32_t)(f.rows[b] | f.prefix[b] << 16 | f.lead[b] << 28);
  r.rep = (int32_t)(f.count | f.step << 16 | f.last << 28);
  return r;
}

static int bad = 0;

static void check(const Fields& f, bool fits, const char* what) {
  const AttnReqBr r = entry(f);
  AttnReqBrPacked p;
  std::memset(&p, 0xA5, sizeof(p));
  if (p.pack(r) != fits) {
    std::printf("%s: packs %d\n", what, !fits);
    ++bad;
    return;
  }
  if (!fits) return;
  const AttnReqBr u = p.unpack();
  if (std::memcmp(&u, &r, sizeof(r)) != 0) {
    std::printf("%s: unpacks to other numbers\n", what);
    ++bad;
  }
}

int main() {
  const Fields zero = {};
  const Fields most = {0xfffff, 4095, 0xfffff, 4095, 0x7fffffff, 0x7fffffff, {1023, 1023, 1023}, {1023, 1023, 1023},
                       {15, 15, 15}, 255, 255, 2};
  check(zero, true, "zero");
  check(most, true, "most");
  struct Limit {
    const char* name;
    uint32_t last;
    std::function<void(Fields&, uint32_t)> set;
  };
  const Limit limits[] = {
      {"q_start", 0xfffff, [](Fields& f, uint32_t v) { f.q_start = v; }},
      {"n", 4095, [](Fields& f, uint32_t v) { f.n = v; }},
      {"ctx", 0xfffff, [](Fields& f, uint32_t v) { f.ctx = v; }},
      {"nv", 4095, [](Fields& f, uint32_t v) { f.nv = v; }},
      {"rows 0", 1023, [](Fields& f, uint32_t v) { f.rows[0] = v; }},
      {"rows 1", 1023, [](Fields& f, uint32_t v) { f.rows[1] = v; }},
      {"rows 2", 1023, [](Fields& f, uint32_t v) { f.rows[2] = v; }},
      {"prefix 0", 1023, [](Fields& f, uint32_t v) { f.prefix[0] = v; }},
      {"prefix 1", 1023, [](Fields& f, uint32_t v) { f.prefix[1] = v; }},
      {"prefix 2", 1023, [](Fields& f, uint32_t v) { f.prefix[2] = v; }},
      {"count", 255, [](Fields& f, uint32_t v) { f.count = v; }},
      {"step", 255, [](Fields& f, uint32_t v) { f.step = v; }},
  };
  for (const Limit& l : limits)
    for (const Fields& base : {zero, most}) {
      Fields f = base;
      for (uint32_t v : {0u, 1u, l.last / 2, l.last}) {
        l.set(f, v);
        check(f, true, l.name);
      }
      l.set(f, l.last + 1);
      check(f, false, l.name);
    }
  for (uint32_t v = 0; v < 16; ++v)  // fields that hold every accepted value
    for (int b = 0; b < 3; ++b) {
      Fields f = most;
      f.lead[b] = v;
      f.last = b;
      check(f, true, "lead, last");
    }
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM), reason="no g++ or no HIP headers")
def test_packed_entries_round_trip(tmp_path):
    src, exe = tmp_path / "packing.cpp", tmp_path / "packing"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", ROCM, "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    got = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert got.returncode == 0, got.stdout
