"""Host-only: every launch of a large call keeps to the runtime's limits (fewer than 2^32 threads in a
dimension, at most 65535 blocks in y and z).  The calls run against a stand-in for hipLaunchKernel that
holds them to these limits; nothing is dereferenced on the host."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = r"""
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim3;
int launches = 0, refused = 0;
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, void* stream) {
  unsigned long long x = (unsigned long long)g.x * b.x, y = (unsigned long long)g.y * b.y, z = (unsigned long long)g.z * b.z;
  int bad = x >> 32 || y >> 32 || z >> 32 || g.y > 65535 || g.z > 65535 || !g.x || !g.y || !g.z || b.x * b.y * b.z > 1024;
  ++launches;
  refused += bad;
  return bad ? 9 : 0;                      /* hipErrorInvalidConfiguration */
}
"""
CALL = r"""
import ctypes as C, json, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
from paper_2510_22049_amd import binding as V
entry, kw = sys.argv[2], json.loads(sys.argv[3])
p, L = C.c_void_p(1 << 20), V.lib()
if entry == "summarize":
    st = L.vista_summarize(C.byref(V.summarize_desc(**kw)), p, p, None, p, p, p, p, p, 1 << 60, None)
elif entry == "attend":
    st = L.vista_target_attend(C.byref(V.AttendDesc(**kw)), p, p, p, None)
else:
    st = L.vista_quantize_summaries(C.byref(V.CodecDesc(**kw)), p, p, p, None)
print(json.dumps([st, C.c_int.in_dll(stub, "launches").value, C.c_int.in_dll(stub, "refused").value]))
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    d = tmp_path_factory.mktemp("stub")
    (d / "stub.c").write_text(STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(d / "stub.so"), str(d / "stub.c")], check=True)
    return str(d / "stub.so")


def call(stub, entry, **kw):
    r = subprocess.run([sys.executable, "-c", CALL, stub, entry, json.dumps(kw)], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout.strip().splitlines()[-1])


# merge: one thread per output element, four where users hold eight records or more
@pytest.mark.parametrize("kw", [
    dict(B=1 << 17, S=256, d=128, H=4, dtype=0, total_items=1 << 20),
    dict(B=1 << 17, S=256, d=128, H=4, dtype=0, total_items=1 << 20, attn=1, self_term=True),
    dict(B=1 << 15, S=512, d=64, H=1, dtype=0, total_items=1 << 24, segment_items=64),
    dict(B=1 << 20, S=100, d=64, H=8, dtype=1, total_items=1 << 20)])
def test_merge_of_many_outputs(stub, kw):
    st, launches, refused = call(stub, "summarize", **kw)
    assert (st, refused) == (0, 0) and launches >= 2


# stage 2 outside the bf16 shapes: a wave for 16 candidates of a head
@pytest.mark.parametrize("kw", [dict(B=1 << 16, C=1 << 15, S=16, d=16, H=1, dtype=1), dict(B=1 << 12, C=1 << 17, S=16, d=64, H=4, dtype=0)])
def test_many_candidates(stub, kw):
    assert call(stub, "attend", **kw) == [0, 1, 0]


# codec: one to eight threads for a (token, head)
@pytest.mark.parametrize("kw", [dict(rows=1 << 28, d=128, H=4, dtype=1), dict(rows=1 << 26, d=512, H=8, dtype=0),
                                dict(rows=(1 << 29) - 32, d=64, H=8, dtype=1)])
def test_many_summary_rows(stub, kw):
    assert call(stub, "quantize", **kw) == [0, 1, 0]
