"""The tree buffer's arrays lie one behind the other, also where a context holds a
few tokens only and every array is rounding: a host program, compiled from the
library's own header and linked with it, asks for the view of every small size and
checks each array against the next and the kernel arguments at the end.  No GPU
call is made.  The same for the segmentation's workspace, where the tables of the
recurrence lie over the distances that the slot scores have read."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2608_07001_amd")

SRC = r"""
#include <stdio.h>
#include <algorithm>
#include <vector>
#include "common.h"
using namespace gkv;
struct Arr { const char* name; const char* p; size_t bytes; };
static int check(const gracekv_config& c) {
  gracekv_plan p;
  if (gracekv_plan_sizes(&c, &p) != GRACEKV_OK) return -1;
  char* base = (char*)0x100000;                 // never dereferenced
  const TreeView v = make_view(base, p);
  const size_t LG = (size_t)c.L * c.G, UC = p.unit_cap, NC = p.node_cap, e = c.dtype == GRACEKV_BF16 ? 2 : 4;
  const int64_t cap = v.long_cap;
  std::vector<Arr> a;
  auto add = [&](const char* n, const void* q, size_t b) { a.push_back({n, (const char*)q, b}); };
  add("sp_E", v.sp_E, NC * 8); add("add_E", v.add_E, UC * 8); add("node_a", v.node_a, NC * 4);
  add("unit_nn", v.unit_nn, UC * 4); add("tok_R", v.tok_R, LG * p.N_c * 4); add("status", v.status, 16);
  add("slots", v.slots, (p.J_cap + 1) * 4); add("work", v.work, UC * 32); add("wctr", v.wctr, 16 * 4);
  add("proto", v.proto, UC * 2 * c.d * e); add("proto_logm", v.proto_logm, UC * 4);
  for (int k = 0; k < LONG_CLASSES; ++k) add("long_items", v.long_items[k], cap * 32);
  add("sub_items", v.sub_items, LG * short_capacity(p.N_c) * 32); add("sub_ctr", v.sub_ctr, LG * 4);
  add("lv_ctr", v.lv_ctr, 16 * 4); add("kargs", v.kargs, KARGS_BYTES);
  if (cap < (int64_t)(LG * (p.N_c / (ST_N + 1)))) { printf("long lists too short\n"); return 1; }
  if (sizeof(Dims) > 512 || sizeof(TreeView) > KARGS_BYTES - 512) { printf("kernel arguments too long\n"); return 1; }
  int bad = 0;
  for (const Arr& x : a)
    if (x.p < base || x.p + x.bytes > base + p.tree_bytes || ((size_t)x.p & 15)) {
      printf("L G %zu N_c %ld: %s outside the buffer or misaligned\n", LG, (long)p.N_c, x.name);
      bad = 1;
    }
  std::stable_sort(a.begin(), a.end(), [](const Arr& x, const Arr& y) { return x.p < y.p; });
  for (size_t i = 0; i + 1 < a.size(); ++i)
    if (a[i].p + a[i].bytes > a[i + 1].p && a[i].bytes && a[i + 1].bytes) {
      printf("L G %zu N_c %ld: %s runs into %s by %zu bytes\n", LG, (long)p.N_c, a[i].name, a[i + 1].name,
             (size_t)(a[i].p + a[i].bytes - a[i + 1].p));
      bad = 1;
    }
  return bad;
}
int main() {
  int seen = 0, bad = 0;
  const int sizes[][2] = {{1, 1}, {2, 1}, {1, 2}, {3, 1}, {2, 2}, {5, 1}, {3, 3}, {16, 8}, {32, 8}, {80, 8}};
  for (auto& s : sizes)
    for (int dt = 0; dt < 2; ++dt)
      for (int64_t N = 1; N <= 700; N += N < 140 ? 1 : 23) {
        gracekv_config c;
        gracekv_default_config(&c);
        c.L = s[0]; c.G = s[1]; c.H = s[1] * 2; c.d = 64; c.n_seg = 1; c.D_hidden = 64; c.W = 3;
        c.dtype = dt; c.N_ctx = N; c.x = N % 3 ? 1.0 : 2.0;
        const int r = check(c);
        seen += r >= 0;
        bad += r > 0;
      }
  printf("%d plans, %d with overlaps\n", seen, bad);
  return bad ? 1 : 0;
}
"""


SEG = r"""
#include <stdio.h>
#include "segment.hip"
using namespace gkv;
int main() {
  int seen = 0, bad = 0;
  for (int64_t N = 1; N < 1100000; N += N < 3000 ? 1 : N / 7 + 1)
    for (int seg = 1; seg <= 3; seg += 2) {
      Dims dm = {};
      dm.N_c = N; dm.T = N + 40; dm.n_seg = seg; dm.Dh = 64; dm.n_min = 16; dm.n_max = 128;
      char* base = (char*)0x100000;               // never dereferenced
      const SegWs s = seg_view(base, dm);
      const int64_t C = dp_chunks(N);
      // what is live together: dist2's last row beside the offsets of all chunks (one chunk: its own only)
      const char* last = (const char*)(s.dist2 + (N - 1) * BAND);
      const char* lo = (const char*)s.dlt;
      const char* hi = C > 1 ? (const char*)(s.cok + C) : (const char*)(s.dlt + 1);
      const bool row = hi <= last || lo >= last + BAND * 4;
      const bool order = (const char*)(s.dlt + C) <= (const char*)s.cdiff && (const char*)(s.cdiff + C) <= (const char*)s.cok &&
                         (const char*)(s.cok + C) <= (const char*)s.bt_ent && (const char*)(s.bt_ent + bt_chunks(N)) <= (const char*)s.bt_tab &&
                         (const char*)(s.bt_tab + bt_chunks(N) * 128) <= (const char*)s.P2;
      const bool ends = (const char*)(s.Fg + C * (DPC + 128)) <= (const char*)s.smax_part &&
                        (const char*)(s.smax_part + N / 16 + 2) <= base + segment_ws_bytes(dm);
      ++seen;
      if (!row || !order || !ends || !seg_tables_fit(s, dm)) {
        if (bad++ < 8) printf("N_c %ld: row %d order %d ends %d check %d\n", (long)N, row, order, ends, (int)seg_tables_fit(s, dm));
      }
    }
  printf("%d sizes, %d wrong\n", seen, bad);
  return bad ? 1 : 0;
}
"""


def _run(tmp_path, name, src, flags):
    (tmp_path / f"{name}.hip").write_text(src)
    exe = str(tmp_path / name)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-std=c++17", "-Xclang",
                    "-target-feature", "-Xclang", "-packed-fp32-ops", "-w", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(PKG, "csrc"), str(tmp_path / f"{name}.hip"), "-o", exe, "-L", PKG,
                    "-l:libgracekv.so", f"-Wl,-rpath,{PKG}"] + flags, check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:]
    return int(r.stdout.split()[0])


def test_arrays_do_not_overlap(tmp_path):
    assert _run(tmp_path, "layout", SRC, ["--offload-host-only", "-O1"]) > 1000


def test_segmentation_tables_leave_live_distances(tmp_path):
    assert _run(tmp_path, "segment_layout", SEG, ["-O1"]) > 5000
