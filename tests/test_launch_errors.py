"""A launch that fails ends its call with GRIFFIN_EHIP, whichever of the call's launches it is.  Nothing runs on a GPU: the
process that makes the calls has the runtime's launch function replaced by one that fails at a chosen launch and else does nothing."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
static int at = -1, count, last;
void shim_fail_at(int i) { at = i; count = 0; last = 0; }
int shim_launches(void) { return count; }
int __hipPushCallConfiguration(void) { return 0; }
int __hipPopCallConfiguration(void) { return 0; }
int hipLaunchKernel(const void *f, ...) { return count++ == at ? (last = 719) : 0; }
int hipGetLastError(void) { int e = last; last = 0; return e; }
int hipGetDevice(int *dev) { *dev = 0; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { return 0; }
"""

CALLS = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1])
import paper_2404_01365_amd as G
FAKE, BIG = 0x7F0000001000, 1 << 40
def layer(gated, d=2048, n=1030, dtype=G.BF16):
    L = G.griffin_layer()
    L.d, L.n, L.dtype, L.act, L.W1, L.W2, L.Wg, L.ld = d, n, dtype, G.ACT_RELU, FAKE, FAKE, FAKE if gated else None, d
    return ctypes.byref(L)
def cu(*v):
    return (ctypes.c_int32 * len(v))(*v)
lib = G.lib
def select(L, tokens):
    return lambda: lib.griffin_prefill_select(L, FAKE, 2048, cu(0, tokens), 1, 500, FAKE, None, None, 0, FAKE, BIG, None)
def phase(L, tokens):
    return lambda: lib.griffin_prompt_phase(L, FAKE, 1032, FAKE, 2048, cu(0, tokens), 1, 500, FAKE, None, FAKE, 2048, FAKE, BIG, None)
calls = {
    'select Eq. 2 in ranges': select(layer(0), 33), 'select Eq. 3 in ranges': select(layer(1), 33),
    'select Eq. 2': select(layer(0), 5000), 'select Eq. 3': select(layer(1), 5000),
    'select fp32': select(layer(1, dtype=G.F32), 40), 'phase': phase(layer(1, n=1032), 700), 'phase fp32': phase(layer(0, n=1032, dtype=G.F32), 40),
    'row': lambda: lib.griffin_ff_decode(layer(1), FAKE, FAKE, 1, FAKE, BIG, None),
    'rows 40': lambda: lib.griffin_ff_decode(layer(1), FAKE, FAKE, 40, FAKE, BIG, None),
    'own sets 40': lambda: lib.griffin_ff_decode_indexed(layer(1), FAKE, 500, 40, FAKE, FAKE, FAKE, BIG, None),
}
for name, call in calls.items():
    shim.shim_fail_at(-1)
    assert call() == G.OK, name
    launches = shim.shim_launches()
    assert launches >= 2, name
    for i in range(launches):
        shim.shim_fail_at(i)
        assert call() == G.EHIP, (name, i)
    print(name, launches)
"""


def test_every_failed_launch_is_reported(tmp_path):
    src, so = str(tmp_path / "shim.c"), str(tmp_path / "shim.so")
    open(src, "w").write(SHIM)
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-O1", src, "-o", so])
    env = dict(os.environ, LD_PRELOAD=":".join(filter(None, [so, os.environ.get("LD_PRELOAD")])), PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", CALLS, so], env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
