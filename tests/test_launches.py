"""What the entry points launch, on the host alone: the library runs in a child process on top
of a stand-in for the HIP runtime that writes launches down instead of running them."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

CHILD = """
import ctypes, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rec.recorder_log.restype = ctypes.c_char_p
sys.path.insert(0, sys.argv[2])
import paper_2406_15486_amd.binding as B
lib = B.load_library()
P = ctypes.c_void_p(0x10000)                 # non-null, 256-aligned, never dereferenced
ref = ctypes.byref
def shape(S, Hq, Hkv=1, batch=1):
    return B._CShape(batch, Hq, Hkv, S, 128, 1, 0.0)
def room(op, sh, n_s=0, chunks=1, blk=1):
    return lib.sa_workspace_bytes(op, ref(sh), ref(B._CSampling(n_s, chunks, blk)))
def strips(S, Hq, Hkv=1, batch=1, ws=None):
    sh = shape(S, Hq, Hkv, batch)
    ws = room(B.SA_OP_SPARSE_ATTN, sh) if ws is None else ws
    assert lib.sa_sparse_attn(ref(sh), P, P, P, P, P, P, P, 4, P, 0, None, None, P, ws, None) == 0
def blocks(S, Hq, Hkv=1, batch=1, blk=128, ws=None):
    sh = shape(S, Hq, Hkv, batch)
    ws = room(B.SA_OP_BLOCK_SPARSE_ATTN, sh, blk=blk) if ws is None else ws
    assert lib.sa_block_sparse_attn(ref(sh), blk, P, P, P, P, P, P, P, 4, P, 0, None, None, P, ws, None) == 0
def sample(S, n_s, Hq, Hkv=1, batch=1, ws=None):
    sh, sm = shape(S, Hq, Hkv, batch), B._CSampling(n_s, 1, 1)
    ws = room(B.SA_OP_SAMPLE_SCORES, sh, n_s) if ws is None else ws
    assert lib.sa_sample_scores(ref(sh), ref(sm), P, P, P, P, None, P, ws, None) == 0
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("recorder") / "hip_recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", os.path.join(HERE, "hip_recorder.cpp"), "-o", so],
                   check=True)
    return so


def _run(recorder, calls):
    """The log of `calls`, a list of (kind, kernel, numbers)."""
    code = CHILD + calls + "\nprint(rec.recorder_log().decode(), end='')\n"
    r = subprocess.run([sys.executable, "-c", code, recorder, ROOT], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [ln.split() for ln in r.stdout.splitlines() if ln.split()[:1] in (["launch"], ["attribute"])]
    assert lines, r.stdout
    return [(kind, name, [int(x) for x in rest]) for kind, name, *rest in lines]


def test_lds_limits_do_not_depend_on_the_call(recorder):
    """A kernel's LDS limit belongs to the whole process: a call that set it to its own need
    could lower it between another thread's setting and launch."""
    log = _run(recorder, "strips(1 << 20, 1); strips(512, 1); blocks(1 << 20, 1); blocks(512, 1); sample(4096, 128, 1)")
    limits = {}
    for kind, name, v in log:
        if kind == "attribute":
            limits.setdefault(name, set()).add(v[1])
    assert any("strip_prep" in n for n in limits) and any("block_prep" in n for n in limits)
    for name, values in limits.items():
        assert len(values) == 1, (name, values)
    for kind, name, v in log:
        if kind == "launch" and v[4] > 0:
            assert v[4] <= max(limits[name]), name


@pytest.mark.parametrize("S,Hq,cut", [(257, 1, False), (512, 1, False), (512, 4, False), (513, 1, True), (768, 8, True),
                                      (1024, 4, True), (2047, 1, True), (2048, 1, True), (3001, 32, False)])
def test_small_problems_are_cut_by_length_whatever_the_path(recorder, S, Hq, cut):
    """Dense, strip and block launches share one rule; up to two query tiles are never cut (a
    second launch costs more than it gives there), and the room is asked for only where they are."""
    calls = f"""
sh = shape({S}, {Hq})
for path in (strips, blocks):
    path({S}, {Hq})
assert lib.sa_dense_attn(ref(sh), P, P, P, P, 0, None, P, room(B.SA_OP_DENSE_ATTN, sh), None) == 0
assert lib.sa_dense_attn_static(ref(sh), P, P, P, P, 0, None, None) == 0
pad = (({S} + 255) // 256) * 256
assert (room(B.SA_OP_DENSE_ATTN, sh) > pad * 256) == {cut}
"""
    log = _run(recorder, calls)
    combined = sum("parts_combine" in name for kind, name, v in log if kind == "launch")
    assert combined == (4 if cut else 0)


# (heads, tokens, core of the dense launch, of swept strips, of swept blocks): below and above the limits
@pytest.mark.parametrize("Hq,S,cores", [(16, 4500, "222"), (8, 9000, "222"), (16, 5100, "222"), (16, 5300, "202"), (16, 6200, "002"), (16, 10000, "002"),
                                        (16, 10300, "000"), (32, 16384, "000"), (32, 1000, "222"), (64, 2100, "202"), (4, 16000, "222")])
def test_core_of_dense_and_swept_tiles_follows_the_launch(recorder, Hq, S, cores):
    """Launches of up to some 1.5 rounds of the CUs are bound by the chain of their heaviest tile, larger ones by
    power: each takes the shape of the MFMAs that is faster there (the results are the same bits)."""
    log = _run(recorder, f"""
sh = shape({S}, {Hq})
assert lib.sa_dense_attn(ref(sh), P, P, P, P, 0, None, P, room(B.SA_OP_DENSE_ATTN, sh), None) == 0
strips({S}, {Hq}); blocks({S}, {Hq})
""")
    flash = [name for kind, name, v in log if kind == "launch" and "12flash_kernel" in name]
    # flash_kernel<mode, fp32 output, blocks in place, parts, core>
    assert [name[:name.index("EEEv")][-1] for name in flash] == list(cores), flash
