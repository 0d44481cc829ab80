"""What a call of the library launches, without a GPU: the call is made in a process whose runtime's launch function only notes the
kernel, its grid and (of the prompt product) its parameters, of a launch on two shapes those of both."""
import ctypes
import json
import os
import re
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_SHIM = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_t;
typedef struct { char name[400]; unsigned grid[3]; unsigned char params[2][144]; } note_t;
static note_t notes[64];
static int count;
int shim_take(void *out) { int n = count; memcpy(out, notes, sizeof(note_t) * n); count = 0; return n; }
static dim3_t grid_of, block_of;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream) { grid_of = grid; block_of = block; return 0; }
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream)
{
    *grid = grid_of; *block = block_of; *lds = 0; *stream = 0;
    return 0;
}
int hipLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream)
{
    Dl_info at;
    note_t *n = &notes[count < 63 ? count++ : 63];
    memset(n, 0, sizeof *n);
    if (dladdr(f, &at) && at.dli_sname)
        strncpy(n->name, at.dli_sname, sizeof n->name - 1);
    n->grid[0] = grid.x; n->grid[1] = grid.y; n->grid[2] = grid.z;
    if (strstr(n->name, "Ff1Params"))
        memcpy(n->params[0], args[0], sizeof n->params[0]);
    if (strstr(n->name, "two_shapes"))
        memcpy(n->params[1], args[1], sizeof n->params[1]);
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipGetDevice(int *dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int dev) { *v = 256; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { return 0; }
"""


class Ff1Params(ctypes.Structure):          # as in csrc/ff1_kernel.h
    _fields_ = ([(p, ctypes.c_void_p) for p in ("X", "Wg", "W1", "bg", "b1", "Z", "rowpart", "Zb")] +
                [(v, ctypes.c_int64) for v in ("ldx", "ldw", "ldz", "ldzb")] +
                [(v, ctypes.c_int32) for v in ("M", "F", "d", "nt", "mt", "splits", "kt_per_split", "kt_per_sum", "z_stream", "rotate", "nt_row")])


class _Note(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char * 400), ("grid", ctypes.c_uint32 * 3), ("params", ctypes.c_ubyte * 144 * 2)]


_FAKE = 0x7F0000001000


def _child():
    import paper_2404_01365_amd as G
    shim = ctypes.CDLL(sys.argv[2])
    notes = (_Note * 64)()
    out = []
    for c in json.load(sys.stdin):
        L = G.griffin_layer()
        L.d, L.n, L.dtype, L.act, L.W1, L.W2, L.ld = c["d"], c["n"], c.get("dtype", G.BF16), c.get("act", G.ACT_SILU), _FAKE, _FAKE, c.get("ld") or c["d"]
        L.Wg = _FAKE if c.get("gated", True) else None
        L.b1 = _FAKE if c.get("bias") else None
        L.bg = _FAKE if c.get("bias") and c.get("gated", True) else None
        cu = [0]
        for v in c["lens"]:
            cu.append(cu[-1] + v)
        cu = (ctypes.c_int32 * len(cu))(*cu)
        S, M, k = len(cu) - 1, cu[len(cu) - 1], max(1, c["n"] // 2)
        ldw = c.get("ldw") or (c["n"] + 7) // 8 * 8

        def call(ws):
            if c["entry"] == "select":       # ldz: rows of a caller's Z that far apart
                return G.lib.griffin_prefill_select(ctypes.byref(L), _FAKE, c["d"], cu, S, k, _FAKE, None, _FAKE if c.get("ldz") else None,
                                                    c.get("ldz") or 0, _FAKE, ws, None)
            if c["entry"] == "phase":
                return G.lib.griffin_prompt_phase(ctypes.byref(L), _FAKE, ldw, _FAKE, c["d"], cu, S, k, _FAKE, None, _FAKE, c["d"], _FAKE, ws, None)
            return G.lib.griffin_ff_prompt_out(_FAKE, c["n"], M, c["n"], c["d"], L.dtype, _FAKE, ldw, None, _FAKE, c["d"], _FAKE, ws, None)

        ws = 1 << 44
        if c.get("least"):                   # the least workspace that is accepted
            lo = 0
            while ws - lo > 256:
                mid = (lo + ws) // 2 // 256 * 256
                lo, ws = (lo, mid) if call(mid) == G.OK else (mid, ws)
        shim.shim_take(notes)
        assert call(ws) == G.OK, c
        found = []
        for i in range(shim.shim_take(notes)):
            p, p2 = ({f: getattr(q, f) or 0 for f, _ in Ff1Params._fields_} for q in (Ff1Params.from_buffer_copy(bytes(b)) for b in notes[i].params))
            found.append(dict(name=notes[i].name.decode(), grid=list(notes[i].grid), second=p2, **p))
        out.append(found)
    json.dump(out, sys.stdout)


def record(calls):
    """calls: dicts of entry ("select", "phase" or "out"), d, n, lens, gated, bias, act, dtype, least, ldz, ld (of the block), ldw (of W2p) -> the launches of each"""
    with tempfile.TemporaryDirectory() as tmp:
        src, so = os.path.join(tmp, "shim.c"), os.path.join(tmp, "shim.so")
        with open(src, "w") as f:
            f.write(_SHIM)
        subprocess.check_call(["gcc", "-shared", "-fPIC", "-O1", src, "-o", so, "-ldl"])
        env = dict(os.environ, LD_PRELOAD=":".join(filter(None, [so, os.environ.get("LD_PRELOAD")])), PYTHONPATH=ROOT)
        r = subprocess.run([sys.executable, os.path.abspath(__file__), "child", so], input=json.dumps(calls), env=env,
                           capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout)


_FORM = re.compile(r"ff1_bf16_mfma_kernelILi(\d)ELb(\d)ELi(\d)ELi(\d)ELb(\d)ELb(\d)ELi(\d)ELb(\d)E")


def form(name):
    """A form of the prompt product's kernel, whatever its activation: "tokens x neurons" of its tiles and what it is for (None: another kernel)."""
    m = _FORM.search(name)
    if not m:
        return None
    _, gated, ti, ni, plain, wide, extra, dual = (int(v) for v in m.groups())
    if plain:
        return "%dx%d raw %s" % (32 * ti, (1 if dual else 2) * 32 * ni, "Eq. 3" if dual else "one matrix")
    if wide:
        return "%dx%d Eq. 2" % (32 * ti, 64 * ni)
    if not gated:
        return "%dx%d Eq. 2 narrow" % (32 * ti, 32 * ni)
    return "%dx%d Eq. 3%s" % (32 * ti, 32 * ni, {0: "", 1: " copy", 2: " biases"}[extra])


_TWO = re.compile(r"ff1_bf16_two_shapes_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)E")


def two_shapes(name):
    """activation, bf16 copy, (tokens, neurons) of the tiles of the first and the second shape (None: another kernel)"""
    m = _TWO.search(name)
    return m and (int(m[1]), m[2] == "1", (32 * int(m[3]), 32 * int(m[4])), (32 * int(m[5]), 32 * int(m[6])))


def route(launch):
    """form, tiles, k-tiles of each (of a range), sums kept apart of a tile"""
    tiles = launch["mt"] * launch["nt"] * launch["splits"]
    kt = min(launch["kt_per_split"], launch["d"] // 64)
    raw = " raw " in form(launch["name"])
    return form(launch["name"]), tiles, kt, 1 if raw else -(-kt // launch["kt_per_sum"])


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    _child()
