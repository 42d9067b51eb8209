"""Which kernels a scoring call launches, on which grid and with which cut: the library's HIP calls go to stand-ins that record names,
grids and arguments, so no GPU is needed. The device is said to have 256 compute units."""
import json
import subprocess
import sys

from test_two_devices_cpu import ROOT, STAND_INS

RECORDING = "#include <string.h>" + STAND_INS.replace("int hipLaunchKernel(const void*, d3, d3, void**, size_t, void*) { return 0; }", r"""
static struct { const void* f; char name[400]; } known[512];
static struct { const char* name; unsigned grid[3]; unsigned threads; size_t lds; int chunk, n_layers, layers_each; } seen[64];
static int n_known, n_seen;
void __hipRegisterFunction(void*, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  int i = 0;
  if (n_known == 512) return;
  for (known[n_known].f = f; name[i] && i < 399; ++i) known[n_known].name[i] = name[i];
  ++n_known;
}
void stand_in_forget() { n_seen = 0; }
int stand_in_launches() { return n_seen; }
const char* stand_in_name(int i) { return seen[i].name; }
long stand_in_value(int i, int what) {
  long v[8] = {seen[i].grid[0], seen[i].grid[1], seen[i].grid[2], seen[i].threads, (long)seen[i].lds, seen[i].chunk, seen[i].n_layers, seen[i].layers_each};
  return v[what];
}
int hipLaunchKernel(const void* f, d3 grid, d3 block, void** args, size_t lds, void*) {
  if (n_seen == 64) return 1;
  auto& s = seen[n_seen++];
  s.name = "?";
  for (int i = 0; i < n_known; ++i) if (known[i].f == f) s.name = known[i].name;
  s.grid[0] = grid.x; s.grid[1] = grid.y; s.grid[2] = grid.z; s.threads = block.x; s.lds = lds;
  if (strstr(s.name, "score_stats_mfma") || strstr(s.name, "score_emit_")) {
    s.chunk = *(int*)args[1]; s.n_layers = *(int*)args[2]; s.layers_each = *(int*)args[3];
  }
  return 0;
}""")

PROGRAM = r"""
import ctypes as C, json, re, sys
stand_ins = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
stand_ins.stand_in_name.restype = C.c_char_p
stand_ins.stand_in_value.restype = C.c_long
from paper_2412_14838_amd import dkv
lib = C.CDLL(dkv.LIB_PATH)
P, I64 = C.c_void_p, C.c_int64
fake, big = P(0x10000), C.c_size_t(1 << 50)
out = []
for L, Hq, Hkv, w, lens, given in json.loads(sys.argv[2]):
    T = sum(lens)
    desc = dkv.make_desc(n_layers=L, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, window=w, pool_kernel=7, layer_max=64, mean_budget=32,
                         interval=1, dtype=dkv.DKV_BF16, n_seqs=len(lens), total_tokens=T, max_seq_len=max(lens))
    stand_ins.stand_in_forget()
    many = (P * L)(*[0x10000] * L)
    strides = I64(128), I64(T * 128)
    if given:
        rc = lib.dkv_score_window_lse_layers(C.byref(desc), 0, L, many, many, *strides, fake, many, fake, fake, big, None)
    else:
        rc = lib.dkv_score_window_layers(C.byref(desc), 0, L, many, many, *strides, fake, fake, fake, big, None)
    assert rc == 0, rc
    sweeps = {}
    for i in range(stand_ins.stand_in_launches()):
        m = re.match(r"_ZN3dkv\d+(score_stats_mfma|score_emit_mfma|score_emit_waves)((?:I|L?i?\d+E|Li\d+E)*)", stand_ins.stand_in_name(i).decode())
        if m:
            v = [stand_ins.stand_in_value(i, k) for k in range(8)]
            sweeps["stats" if "stats" in m.group(1) else "emit"] = {
                "kernel": m.group(1), "template": [int(x) for x in re.findall(r"Li(\d+)E", m.group(2))], "grid": v[:3], "threads": v[3],
                "lds": v[4], "chunk": v[5], "layers": v[6], "layers_each": v[7]}
    out.append(sweeps)
print(json.dumps(out))
"""


def sweeps(tmp_path, calls):
    """calls: (layers, query heads, KV heads, window, lengths, normalisers handed over) each, bf16, head size 128, pooling 7. Per call
    {"stats": .., "emit": ..} with the kernel's name and template arguments, grid, threads, dynamic LDS, chunk, layers, layers_each."""
    src, lib = tmp_path / "stand_ins.cpp", tmp_path / "libstand_ins.so"
    src.write_text(RECORDING)
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    run = subprocess.run([sys.executable, "-c", PROGRAM, str(lib), json.dumps(calls)], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert run.returncode == 0, run.stderr
    return json.loads(run.stdout.strip().splitlines()[-1])
