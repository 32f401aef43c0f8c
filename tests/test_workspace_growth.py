"""A workspace whose growth fails (E_NOMEM) leaves no pointer to freed memory and
no capacity that a later, smaller call would trust.

The failure is forced on the host, by a size no device has (or, without a
device, by any size): no GPU is needed."""
import os
import subprocess

import pytest

from paper_2608_11249_amd import build

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "runtime.h"

static bool owned(const dlmc_model& m, const void* p) {
  return !p || std::find(m.allocs.begin(), m.allocs.end(), p) != m.allocs.end();
}

int main() {
  dlmc_model m;
  m.cfg.max_batch = 4096;
  m.cfg.vocab = 0x7ffffffe;
  // buffers of an earlier, smaller call: not in allocs, as after their free
  int mark = 0;
  void* old = &mark;
  m.sel_pos = m.sel_row = m.n_sel = m.dec = m.slot_rows = m.tokens_dev = (int32_t*)old;
  m.cdf = m.sym = (uint32_t*)old;
  m.cdf_ws = old;
  m.slot_base = (int64_t*)old;
  m.slot_mx = (float*)old;
  m.sel_cap = 8;
  m.tokens_cap = 8;
  int failed = 0;
  try { m.ensure_sel(1 << 16); } catch (const dlmc::Error& e) { failed += e.code == DLMC_E_NOMEM; }
  try { m.ensure_tokens((size_t)1 << 50); } catch (const dlmc::Error& e) { failed += e.code == DLMC_E_NOMEM; }
  bool ok = failed == 2 && m.sel_cap == 0 && m.tokens_cap == 0;
  for (const void* p : {(void*)m.sel_pos, (void*)m.sel_row, (void*)m.n_sel, (void*)m.dec,
                        (void*)m.slot_rows, (void*)m.tokens_dev, (void*)m.cdf, (void*)m.sym,
                        m.cdf_ws, (void*)m.slot_base, (void*)m.slot_mx})
    ok = ok && owned(m, p);
  std::printf("%s failed %d sel_cap %d tokens_cap %zu\n", ok ? "ok" : "stale", failed, m.sel_cap,
              m.tokens_cap);
  return ok ? 0 : 1;
}
"""


def test_failed_growth_leaves_nothing_stale(tmp_path):
    lib = build.OUT
    if not os.path.exists(lib):
        pytest.skip("the library is not built")
    src, obj, exe = (tmp_path / n for n in ("growth.cpp", "growth.o", "growth"))
    src.write_text(PROGRAM)
    # host code, with the compiler and flags of the library's own (one ABI)
    subprocess.run([build.HIPCC, *build.COMMON, "-I", build.CSRC, "-c", str(src), "-o", str(obj)],
                   check=True, timeout=120)
    subprocess.run([build.HIPCC, str(obj), lib, "-Wl,-rpath," + os.path.dirname(lib), "-o", str(exe)],
                   check=True, timeout=120)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
