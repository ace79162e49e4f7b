"""What the library enqueues, without a GPU: the calls go to tests/hip_recorder.c in place of the
HIP runtime (in a child process), and the order that streams and events give the launches is
worked out from what it wrote down."""
import ctypes as C
import json
import math
import os
import random
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN, AUX = 0xa0, 0xb0                                 # streams; like every address here never dereferenced
F32, BF16 = 0, 1


def _child(recorder, library, calls):
    rec = C.CDLL(recorder, mode=C.RTLD_GLOBAL)         # found before the runtime that the library is linked with
    lib = C.CDLL(library)
    rec.recorder_text.restype = C.c_char_p
    P = lambda i: C.c_void_p(0x100000000000 + (i << 40))  # noqa: E731 (buffers far apart)
    out = []
    for c in calls:
        rec.recorder_reset()
        if c["what"] == "layer":
            desc = (C.c_int32 * 10)(*[c[n] for n in ("T", "d", "F", "E", "k", "capacity", "dtype")], 0, 0, c["cg"])
            w = (C.c_int64 * 13)(*[P(20 + i).value for i in range(11)], 0, 0)
            size = C.c_size_t(0)
            assert lib.scmoe_workspace_bytes(desc, C.byref(size)) == 0
            st = lib.scmoe_layer_forward(desc, P(1), C.c_int64(c["d"]), P(2), C.c_int64(c["d"]), w, P(3) if c["res"] else None,
                                         C.c_int64(c["d"]), P(4), C.c_int64(c["d"]), None, P(5), size, C.c_void_p(MAIN),
                                         C.c_void_p(AUX) if c["two"] else None)
        elif c["what"] == "ffn":
            n, d, F, code = c["T"], c["d"], c["F"], c["dtype"]
            st = lib.scmoe_expert_ffn(P(1), C.c_int64(d), code, P(2), n, c["E"], d, F, P(3), C.c_int64(d), None, P(4), C.c_int64(F),
                                      None, P(5), C.c_int64(F), P(6), C.c_int64(d), 0, None, C.c_size_t(0), C.c_void_p(MAIN))
        elif c["what"] == "gate":
            st = lib.scmoe_gate_topk(P(1), C.c_int64(c["d"]), c["dtype"], C.c_void_p(P(2).value + c["off"]), None, c["T"], c["d"], c["E"],
                                     c["k"], 0, P(3), P(4), P(5), C.c_void_p(MAIN))
        out.append([st, rec.recorder_text().decode()])
    print(json.dumps(out))


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    """record(calls) -> for each call its status and the lines of the recorder, split into words."""
    so = str(tmp_path_factory.mktemp("recorder") / "hip_recorder.so")
    subprocess.check_call(["gcc", "-std=c11", "-O1", "-Wall", "-shared", "-fPIC", os.path.join(ROOT, "tests", "hip_recorder.c"),
                           "-o", so])
    library = os.path.join(ROOT, "paper_2404_05019_amd", "libscmoe.so")

    def run(calls):
        r = subprocess.run([sys.executable, os.path.abspath(__file__), so, library, json.dumps(calls)], stdout=subprocess.PIPE,
                           stderr=subprocess.PIPE, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-3000:]
        return [(st, [line.split(" ") for line in text.splitlines()]) for st, text in json.loads(r.stdout)]
    return run


def _order(lines):
    """(kernels, after, end): for each launch its name, stream and the launches that are done before it
    starts; the launches that are done before anything enqueued later on the main stream."""
    kernels, done, events = [], {}, {}
    for w in lines:
        if w[0] == "kernel":
            stream = int(w[1], 16)
            kernels.append((w[2], stream, frozenset(done.get(stream, set()))))
            done.setdefault(stream, set()).add(len(kernels) - 1)
        elif w[0] == "record":
            events[w[2]] = set(done.get(int(w[1], 16), set()))
        elif w[0] == "wait":
            done.setdefault(int(w[1], 16), set()).update(events.get(w[2], set()))
    return kernels, done.get(MAIN, set())


def _at(kernels, part):
    return [i for i, k in enumerate(kernels) if part in k[0]]


def _layers():
    out = []
    for dtype, T, d, F in [(F32, 256, 64, 256), (BF16, 8, 256, 512), (BF16, 4000, 512, 2048), (BF16, 300, 72, 200),
                           (BF16, 64, 1024, 4096)]:
        for k in (1, 2):
            for cg in (0, 1, 2):
                for res in (False, True):
                    for capacity in (T * k, 10, 0):
                        out.append(dict(what="layer", T=T, d=d, F=F, E=8, k=k, capacity=capacity, dtype=dtype, cg=cg, res=res,
                                        two=True))
    return out


def test_second_stream_of_a_layer_is_ordered_with_the_first(record):
    """Both streams of a layer call: nothing of the call starts before what the main stream held, the
    coefficients are written before they are read, the decode that adds to the shared expert's rows
    comes after them, and at the end the main stream waits for everything."""
    calls = _layers()
    for c, (st, lines) in zip(calls, record(calls)):
        assert st == 0, c
        kernels, end = _order(lines)
        assert {s for _, s, _ in kernels} == {MAIN, AUX}, c
        assert end == set(range(len(kernels))), c
        aux = {i for i, k in enumerate(kernels) if k[1] == AUX}
        coef = _at(kernels, "coef_gate_kernel")
        assert len(coef) == (1 if c["cg"] else 0)
        for name in ("scale_gate", "combine_kernel"):
            for i in _at(kernels, name):
                assert set(coef) <= kernels[i][2], (c, name)
        if c["capacity"]:                              # (otherwise no decode: nothing is kept)
            last = kernels[max(i for i, k in enumerate(kernels) if k[1] == MAIN)]
            assert aux <= last[2], c


def _layer(T, d, F, E=8, k=1, dtype=BF16, two=False):
    return dict(what="layer", T=T, d=d, F=F, E=E, k=k, capacity=T * k, dtype=dtype, cg=0, res=False, two=two)


def test_small_products_take_the_direct_kernel_and_many_rows_the_tiled_one(record):
    """bf16: both limits of the rule (multiply-adds per product, outputs per call), and what it leaves out."""
    ffn = dict(what="ffn", E=8, dtype=BF16)
    direct = [_layer(256, 256, 1024), _layer(400, 512, 2048), _layer(4000, 64, 128), _layer(30000, 64, 64), dict(ffn, T=8000, d=64, F=192),
              _layer(8, 2048, 8192, 16), _layer(2000, 256, 1024, dtype=F32)]
    tiled = [_layer(30000, 64, 128), _layer(30000, 64, 256, two=True), _layer(2000, 256, 512), _layer(1000, 512, 2048),
             dict(ffn, T=32768, d=64, F=192), dict(ffn, T=500, d=1024, F=1024)]
    for want, calls in (("gemm_direct_kernel", direct), ("gemm_bf16_kernel", tiled)):
        for c, (st, lines) in zip(calls, record(calls)):
            kernels, _ = _order(lines)
            gemms = _at(kernels, "gemm_")
            assert st == 0 and gemms and _at(kernels, want) == gemms, c


def test_tiled_chains_of_the_test_helper_is_the_library_s_rule(record):
    """The rule as gpu_util states it for the GPU tests, against the kernels the library launches."""
    from gpu_util import tiled_chains
    rng = random.Random(3)
    calls = []
    for _ in range(300):
        T, E = int(math.exp(rng.uniform(0, math.log(40000)))), rng.choice([1, 2, 4, 8, 16, 64])
        d, F = (rng.choice([64, 64, 128, 256, 512, 1024, 2048]) for _ in range(2))
        calls.append(_layer(T, d, F, E, rng.randint(1, min(E, 4))))
        calls[-1]["capacity"] = rng.choice([10, max(1, T // E), T * calls[-1]["k"]])
    seen = set()
    for c, (st, lines) in zip(calls, record(calls)):
        kernels, _ = _order(lines)
        ran = {n for n in ("gemm_bf16_kernel", "gemm_direct_kernel") if _at(kernels, n)}
        want = tiled_chains(c["T"], c["d"], c["F"], c["E"], c["k"], c["capacity"])
        assert st == 0 and ran == {"gemm_bf16_kernel" if t else "gemm_direct_kernel" for t in want}, c
        seen.add(want)
    assert seen >= {(False, False), (True, True), (True, False)}


def test_joint_second_gemm_only_where_its_rule_and_its_forms_allow_it(record):
    """Top-1 layers on one stream: two GEMM launches where the second products are one, else three."""
    base = _layer(16384, 1024, 4096)
    joint = [base, dict(base, res=True), dict(base, capacity=100), _layer(30000, 768, 3072), _layer(16384, 1024, 4096, 32),
             _layer(4096, 2048, 128, 16)]
    apart = [dict(base, two=True), dict(base, cg=1), dict(base, cg=2, res=True), _layer(32768, 2048, 8192, 16),    # k-tiles of padding
             _layer(16384, 1024, 4096 + 64), _layer(140000, 256, 512), _layer(8192, 1024, 4096, 8)]   # odd, dispatch in three launches, few tiles
    for want, calls in ((2, joint), (3, apart)):
        for c, (st, lines) in zip(calls, record(calls)):
            kernels, _ = _order(lines)
            gemms = _at(kernels, "gemm_")
            assert st == 0 and len(gemms) == (4 if c["two"] else want) and gemms == _at(kernels, "gemm_bf16_kernel"), c


def test_joint_second_gemm_needs_rows_for_its_tiles(record):
    """Experts of fewer than 256 rows: the shared expert's product would get a tile per expert as well, which
    pays up to 0.4 tiles of 256 x 256 per compute unit more than it has alone."""
    apart = [_layer(T, 1024, 2048, 64) for T in (1100, 1500, 2000, 4200, 8192, 9800)] + [_layer(T, 2048, 2048, 32) for T in (600, 1000, 4096)]
    apart += [dict(_layer(16384, 1024, 4096, 32), capacity=26), _layer(4200, 1024, 2048, 48), _layer(2100, 2048, 2048, 24)]
    joint = [_layer(T, 1024, 2048, 64) for T in (10000, 16384)] + [_layer(T, 2048, 2048, 32) for T in (5120, 8192)]
    joint += [dict(_layer(T, 2048, F, E), capacity=cap, res=cap == 260) for T, F, E, cap in              # (what the GPU tests rely on)
              [(4200, 128, 16, 4200), (4200, 384, 16, 150), (4200, 1024, 16, 260), (5200, 1152, 12, 1)]]
    joint += [dict(_layer(16400, 1024, 256, 4), capacity=3000), dict(_layer(3900, 2304, 2048, 14), capacity=200)]
    joint += [dict(_layer(16384, 1024, 4096, 32), capacity=60), _layer(6000, 1024, 1024, 48), _layer(4096, 2048, 2048, 24)]
    for want, calls in ((2, joint), (3, apart)):
        for c, (st, lines) in zip(calls, record(calls)):
            kernels, _ = _order(lines)
            gemms = _at(kernels, "gemm_bf16_kernel")
            assert st == 0 and len(gemms) == want, (c, [k[0] for k in kernels])


def _direct_shapes(lines):
    """(fp32, row subtiles, column subtiles, ring slots; 0: what fits, -1: no ring) of the direct kernel's launches."""
    names = [w[2] for w in lines if w[0] == "kernel" and "gemm_direct_kernel" in w[2]]
    return [tuple(int(v.replace("n", "-")) for v in re.search(r"gemm_direct_kernelILb(\d)ELi(\d)ELi(\d)ELi(n?\d)E", n).groups())
            for n in names]


def test_tile_shapes_of_the_direct_kernel(record):
    """Which calls take which tiles; the GPU tests of a shape rely on it (calls with 16 rows and a K of 128 steps: 16 x 16)."""
    ffn = lambda T, E, d, F, dtype=BF16: dict(what="ffn", T=T, E=E, d=d, F=F, dtype=dtype)  # noqa: E731
    short, long, few = (0, 1, 2, 3), (0, 1, 2, 0), (0, 1, 1, 0)      # 16 x 32 for a short and for a longer K; 16 x 16
    want = [(ffn(16, 4, 64, 4160), [short, few]), (ffn(16, 1, 128, 4096), [long, few]), (ffn(8, 2, 4160, 4096), [few, few]),
            (_layer(8, 256, 4096, 16), [short, few]), (_layer(1, 64, 8192, 4), [long, few]), (_layer(8, 2048, 8192, 16), [long, few]),
            (ffn(18, 4, 64, 4160), [short, long]),                                 # two rows more
            (ffn(32, 32, 512, 1024), [short, short]), (ffn(64, 64, 512, 1024), [(0, 2, 2, 2)] * 2),
            (_layer(2048, 384, 1536, dtype=F32), [(1, 2, 2, 2), (1, 4, 4, -1)]), (_layer(64, 1024, 4096, dtype=F32), [(1, 2, 2, 0), (1, 2, 1, 0)]),
            # fp32, K of 40 steps: 32 x 32 while 64 x 64 tiles are few (8 per compute unit; 20); of 24 always
            (_layer(3000, 640, 1280, dtype=F32), [(1, 2, 2, 2), (1, 4, 4, -1)]), (_layer(8000, 640, 1280, dtype=F32), [(1, 4, 4, -1)] * 2),
            (_layer(20000, 384, 768, dtype=F32), [(1, 2, 2, 2), (1, 4, 4, -1)]),
            # fp32, one product alone: registers below 10 rows per segment
            (ffn(40, 16, 768, 3072, F32), [(1, 2, 2, -1), (1, 2, 1, -1)]), (ffn(200, 16, 1024, 4096, F32), [(1, 2, 2, 0), (1, 2, 1, 0)]),
            (ffn(120, 8, 1024, 4096, F32), [(1, 2, 2, 0), (1, 2, 1, 0)]),
            # rows that do not begin at 128-byte lines (72, 200, 1032, 4104, 4120 columns ...): no ring
            (ffn(1, 1, 72, 4096), [(0, 1, 2, -1), few]), (ffn(16, 2, 200, 4104), [(0, 1, 2, -1), (0, 1, 1, -1)]),
            (ffn(16, 16, 1032, 4096), [(0, 1, 2, -1), few]), (ffn(16, 3, 4120, 72), [(0, 1, 1, -1), (0, 1, 2, -1)]),
            (_layer(16, 136, 4104, 5), [(0, 1, 2, -1), (0, 1, 1, -1)]), (_layer(300, 776, 2072, 32), [(0, 2, 2, -1)] * 2),
            (ffn(2000, 2, 136, 776), [(0, 4, 4, -1), (0, 2, 2, -1)]), (ffn(18, 2, 72, 2120, F32), [(1, 2, 2, -1), (1, 2, 1, -1)]),
            (_layer(100, 1000, 2664, dtype=F32), [(1, 2, 2, -1), (1, 2, 1, -1)]),
            (ffn(2040, 3, 72, 1000, F32), [(1, 2, 2, 2), (1, 2, 2, 0)])]           # fp32, 128 rows per segment: rings all the same
    got = [(c, _direct_shapes(lines)) for (c, _), (st, lines) in zip(want, record([c for c, _ in want]))]
    assert got == want, "\n".join(str(g) for g in got)


def test_gate_kernels(record):
    """The matrix-core kernel wherever W_g is 16-byte aligned; else one lane per chain up to 65536 lanes."""
    gate = lambda T, d, E, off, dtype=F32, k=1: dict(what="gate", T=T, d=d, E=E, off=off, dtype=dtype, k=k)  # noqa: E731
    want = [(gate(40, 264, 5, 4), "gate_small_kernel"), (gate(100, 72, 40, 4, BF16, 4), "gate_small_kernel"),
            (gate(1024, 40, 64, 8), "gate_small_kernel"), (gate(1025, 40, 64, 12), "gate_kernel"), (gate(70000, 72, 8, 4), "gate_kernel")]
    want += [(dict(c, off=0), "gate_mfma_kernel") for c, _ in want]
    for (c, name), (st, lines) in zip(want, record([c for c, _ in want])):
        kernels = [w[2] for w in lines if w[0] == "kernel"]
        assert st == 0 and len(kernels) == 1 and "%d%s" % (len(name), name) in kernels[0], (c, kernels)


def test_first_gemm_of_small_tiles_where_the_large_ones_leave_a_round_partly_empty(record):
    """128 x 128 tiles in a first GEMM of 129 to 320 rows per segment: not where the large tiles fit one round, nor
    where they nearly fill the second."""
    lay = lambda T, d, F, E, k=1: dict(_layer(T, d, F, E, k), capacity=-(-5 * k * T // (4 * E)))  # noqa: E731
    small = [lay(4000, 640, 1728, 24), lay(1302, 512, 2048, 32, 4), lay(2500, 768, 3072, 16), lay(2000, 512, 2048, 32, 4)]
    large = [lay(2500, 2048, 2048, 16), lay(1302, 512, 1344, 32, 4), lay(1700, 512, 1344, 32, 4), lay(1200, 1024, 4096, 8),
             lay(2500, 1024, 4096, 16), lay(16384, 1024, 4096, 8), lay(6400, 768, 2048, 32)]
    for edge, calls in ((128, small), (256, large)):
        for c, (st, lines) in zip(calls, record(calls)):
            first = next(w[2] for w in lines if w[0] == "kernel" and "gemm_bf16_kernel" in w[2])
            assert st == 0 and "TileCfgILi%dE" % edge in first, (c, first)


def test_first_gemm_alone_of_large_tiles_that_fill_a_round(record):
    """256 x 256 tiles in a first GEMM without the shared expert: four fifths of a round and more, 85 % full in both directions."""
    ffn = lambda T, d, F, E: dict(what="ffn", T=T, d=d, F=F, E=E, dtype=BF16)  # noqa: E731
    large = [ffn(8192, 384, 1536, 8), ffn(6000, 512, 2048, 8), ffn(16451, 192, 768, 12)]
    small = [ffn(15212, 320, 640, 8), ffn(15134, 384, 768, 8), ffn(21226, 128, 320, 8), ffn(23447, 128, 320, 4), ffn(5000, 512, 2048, 12)]
    for edge, calls in ((256, large), (128, small)):
        for c, (st, lines) in zip(calls, record(calls)):
            first = next(w[2] for w in lines if w[0] == "kernel" and "gemm_bf16_kernel" in w[2])
            assert st == 0 and "TileCfgILi%dE" % edge in first, (c, first)


def test_second_gemm_of_wide_tiles_and_second_gemms_in_one_launch(record):
    """256 x 128 tiles of 16 k-tiles and more in up to a round or from 1.75 on; both second GEMMs of a top-1 layer in one launch
    where that saves a partly filled round (what the GPU tests of those tiles rely on is among the calls)."""
    from test_gpu_parity import WIDE_FFN, WIDE_LAYERS
    ffn = [dict(what="ffn", E=E, T=sum(lens) + extra, d=d, F=F, dtype=BF16) for E, lens, d, F, extra in WIDE_FFN]
    lay = [dict(_layer(T, d, F, E, k, two=two), capacity=C_, cg=cg, res=res) for T, d, F, E, k, C_, cg, res, two, shared in WIDE_LAYERS if shared]
    wide = [(c, 1) for c in ffn + lay[:2]] + [(lay[2], 2), (_layer(3001, 768, 3072, 12, 2), 1), (_layer(6000, 512, 2048), 1), (_layer(9000, 768, 3072), 2),
                                              (_layer(6000, 1024, 4096), 2), (_layer(8192, 1024, 4096), 1), (_layer(1664, 1216, 4864, 16), 1), (_layer(654, 1984, 3968, 12, 2), 1)]
    other = [_layer(16384, 1024, 4096), _layer(32000, 128, 512), _layer(12000, 768, 2048), dict(what="ffn", E=16, T=8192, d=1024, F=4096, dtype=BF16),
             _layer(500, 2048, 8192, 16), _layer(18538, 576, 1536, 12), _layer(17279, 192, 768, 16), _layer(6780, 320, 640, 2), _layer(4999, 768, 2048, 8),
             dict(what="ffn", E=32, T=10708, d=768, F=2048, dtype=BF16), dict(what="ffn", E=8, T=21385, d=320, F=1280, dtype=BF16),
             _layer(1204, 1984, 3968, 16), _layer(1641, 1088, 4352, 32, 2)]
    for c, (st, lines) in zip([c for c, _ in wide], record([c for c, _ in wide])):
        kernels, _ = _order(lines)
        n = sum("TileCfgILi256ELi128E" in k[0] for k in kernels)
        assert st == 0 and n == dict((id(a), b) for a, b in wide)[id(c)], (c, [k[0] for k in kernels])
    for c, (st, lines) in zip(other, record(other)):
        kernels, _ = _order(lines)
        assert st == 0 and not any("TileCfgILi256ELi128E" in k[0] for k in kernels), (c, [k[0] for k in kernels])


def test_second_gemm_of_short_tiles(record):
    """64 x 128 tiles up to 53 rows per expert, 3/8 to 1 or 5/4 to 2 of them per CU, and no other second GEMM beside them; both
    second GEMMs of a top-1 layer in one launch of at most two tiles per CU."""
    from test_gpu_parity import SHORT_FFN, SHORT_LAYERS
    calls = [dict(what="ffn", E=E, T=sum(lens), d=d, F=F, dtype=BF16) for E, lens, d, F in SHORT_FFN]
    calls += [dict(_layer(T, d, F, E, k, two=two), capacity=C_, cg=cg, res=res) for T, d, F, E, k, C_, cg, res, two in SHORT_LAYERS]
    calls += [_layer(500, 2048, 8192, 16), _layer(400, 1024, 2048, 17)]
    for c, (st, lines) in zip(calls, record(calls)):
        kernels, _ = _order(lines)
        n = sum("TileCfgILi64ELi128E" in k[0] for k in kernels)
        assert st == 0 and n == 1 and len(_at(kernels, "combine_kernel")) == (c["what"] == "layer" and not c["two"]), (c, [k[0] for k in kernels])
    cut = [_layer(86, 2048, 5440, 4, 2), _layer(182, 1536, 6144, 4)]       # a long K, 128-row tiles too many to be cut
    for c, (st, lines) in zip(cut, record(cut)):
        assert st == 0 and sum("TileCfgILi64ELi128E" in k[0] for k in _order(lines)[0]) == 1, c
    other = [_layer(39, 1472, 3904, 4, 4), _layer(1500, 1024, 4096, 16), _layer(8, 2048, 8192, 16), _layer(600, 1536, 4096, 12), _layer(224, 1728, 4608, 16, 2), _layer(400, 1024, 2048, 24),
             _layer(64, 1280, 2560, 8, 4), _layer(99, 1600, 6400, 8, 3, two=True), _layer(265, 1344, 3584, 16, 2), _layer(600, 2048, 2048, 32),
             dict(what="ffn", E=16, T=940, d=1984, F=5312, dtype=BF16), dict(what="ffn", E=4, T=126, d=1472, F=3904, dtype=BF16)]
    for c, (st, lines) in zip(other, record(other)):
        assert st == 0 and not any("TileCfgILi64ELi128E" in k[0] for k in _order(lines)[0]), c


def test_dropped_rows_under_a_coefficient_gate_are_not_left_to_the_combine_kernel(record):
    """It would scale the shared expert's rounded rows and round a second time; with a residual, without drops or without
    the gate it rounds as often as the two decodes do."""
    base = dict(_layer(2364, 1152, 2304), cg=1, capacity=370)
    few = dict(_layer(300, 1088, 2112, 16), cg=1, capacity=25)
    for want, calls in ((0, [base, dict(base, cg=2), few]),
                        (1, [dict(base, cg=0), dict(base, res=True), dict(base, capacity=2364), dict(few, cg=0), dict(few, res=True), dict(few, capacity=300)])):
        for c, (st, lines) in zip(calls, record(calls)):
            kernels, _ = _order(lines)
            assert st == 0 and len(_at(kernels, "combine_kernel")) == want, (c, [k[0] for k in kernels])


def test_gate_on_the_side_of_the_shared_expert_s_first_gemm(record):
    """No launch of gate, encode and coefficient gate where the first of three products' launches does them, which is where the
    shared expert's tiles apart from the routed ones take no round more (the GPU tests rely on the first ones)."""
    from test_gpu_parity import LONG_SIDE_LAYERS, SIDE_LAYERS
    side = [dict(_layer(T, d, F, E, k), capacity=C_, cg=cg, res=res) for T, d, F, E, k, C_, cg, res in SIDE_LAYERS + LONG_SIDE_LAYERS]
    side += [_layer(500, 2048, 8192, 16), dict(_layer(8192, 384, 1536), capacity=1280), _layer(6000, 512, 2048)]
    apart = [_layer(500, 2048, 8192, 16, two=True), _layer(500, 2048, 8192, 24), _layer(16384, 1024, 4096), _layer(1500, 1536, 4096),
             _layer(3001, 768, 3072, 12, 2), _layer(8000, 192, 768), _layer(8, 2048, 8192, 16), _layer(20000, 512, 2048, k=2)]
    apart += [dict(_layer(T, 256, F), cg=cg) for T in (16385, 32768) for F in (128, 256) for cg in (0, 2)]      # (more gate workgroups than CUs)
    for want, calls in ((True, side), (False, apart)):
        for c, (st, lines) in zip(calls, record(calls)):
            kernels, _ = _order(lines)
            first = next(k[0] for k in kernels if "gemm_" in k[0])
            assert st == 0 and ("ELb1ELi1EEE" in first) == want, (c, [k[0] for k in kernels])
            assert (not any(n in k[0] for k in kernels for n in ("gate_mfma_kernel", "dispatch_", "coef_gate_kernel"))) == want, c


def test_gate_on_the_side_not_where_it_ends_later_or_a_round_is_lost(record):
    """The encode by one workgroup has as many turns as the tiles have k-tiles (three times as many at 256 rows), and the routed
    experts' launch has no round more, also at a skewed load; capacities that drop rows leave the joint launch with fewer."""
    lay = lambda T, d, F, E, k=1, cap=None, cg=0: dict(_layer(T, d, F, E, k), capacity=T if cap is None else cap, cg=cg)  # noqa: E731
    side = [lay(512, 256, 4096, 5, 2, 120), lay(8192, 384, 1536, 8, 1, 1280), lay(7883, 512, 1344, 8, 1, 1232), lay(4018, 576, 2304, 8), lay(3418, 512, 1344, 16, 2, 535, 2)]
    apart = [lay(513, 256, 4096, 5, 2, 120), lay(5161, 256, 704, 8, 2), lay(3305, 256, 704, 8, 4, 2066, 1), lay(2304, 384, 768, 4, 4, 2880),
             lay(7809, 384, 1024, 8, 4, 3905, 1), lay(2733, 1920, 3840, 16), lay(8205, 384, 1024, 4, 1, 2565), lay(1500, 1536, 4096, 8),
             lay(3418, 512, 1344, 16, 2, 535), lay(1828, 960, 3840, 8), lay(6950, 768, 1536, 8, 2, 2172, 1), lay(2622, 1984, 3968, 16, 3)]
    for want, calls in ((True, side), (False, apart)):
        for c, (st, lines) in zip(calls, record(calls)):
            kernels, _ = _order(lines)
            assert st == 0 and any("ELb1ELi1EEE" in k[0] for k in kernels) == want, (c, [k[0] for k in kernels])


def test_second_gemms_of_a_layer_in_one_launch_up_to_two_rounds_from_above(record):
    """Not where both would need a third round of 256 x 128 tiles, with the experts' last row tiles counted from above."""
    one = [_layer(1500, 1536, 4096), _layer(2048, 512, 2048), _layer(3300, 1280, 4096), _layer(1024, 1024, 2048)]
    two = [_layer(20387, 320, 1280, 16), _layer(14602, 512, 1344, 24), _layer(10491, 640, 2560, 32), _layer(2117, 2048, 4096), _layer(2421, 1856, 4928)]
    for want, calls in ((1, one), (2, two)):
        for c, (st, lines) in zip(calls, record(calls)):
            kernels, _ = _order(lines)
            assert st == 0 and len([k for k in kernels if "gemm_bf16" in k[0] and "EEELb0E" in k[0]]) == want, (c, [k[0] for k in kernels])
            assert len(_at(kernels, "combine_kernel")) == (want == 1), c


def test_gate_workgroups_on_the_side_have_no_tile(record):
    """Every XCD's tiles go to its first workgroups and the gate's are the launch's last ones: room for both, whatever the
    remainders of the tiles and of the gate's workgroups by eight are."""
    rng = random.Random(7)
    calls = [_layer(7883, 512, 1344), _layer(3712, 1344, 3584), dict(_layer(1480, 1920, 7680), cg=1)]
    calls += [dict(_layer(int(math.exp(rng.uniform(math.log(300), math.log(9000)))), 64 * rng.randint(4, 32), 64 * rng.randint(10, 128),
                          rng.choice([2, 4, 8, 12, 16]), rng.choice([1, 1, 2])), cg=rng.choice([0, 1])) for _ in range(400)]
    seen = set()
    for c, (st, lines) in zip(calls, record(calls)):
        assert st == 0
        first = next((w for w in lines if w[0] == "kernel" and "gemm_bf16_kernel" in w[2]), None)
        if first is None or "ELb1ELi1EEE" not in first[2]:
            continue
        edge = int(re.search(r"TileCfgILi(\d+)E", first[2]).group(1))
        tiles, gate = -(-c["T"] // edge) * -(-c["F"] // edge), -(-c["T"] // (edge // 2))
        assert int(first[3]) >= -(-tiles // 8) * 8 + gate, (c, first[2:5])
        seen.add((edge, tiles % 8 > 0))
    assert len(seen) == 4


def test_no_launch_passes_the_limit_on_work_items(record):
    """2^32 work-items in x is what the runtime takes; 1.1 million rows of 65544 columns need more
    workgroups than that (144 GB of hidden rows in bf16: they fit the card)."""
    calls = [dict(what="ffn", E=E, T=T, d=d, F=F, dtype=BF16) for E, T, d, F in
             [(1, 1100000, 8, 65544), (8, 1100000, 72, 65544), (1, 300, 72, 200), (2, 600000, 120120, 8)]]
    for c, (st, lines) in zip(calls, record(calls)):
        gemms = [w for w in lines if w[0] == "kernel" and "gemm_direct_kernel" in w[2]]
        assert st == 0 and len(gemms) == 2, c
        for w, width in zip(gemms, (c["F"], c["d"])):
            gx, gy, gz, bx = (int(v) for v in w[3:7])
            assert gx * bx < 2 ** 32 and gy < 65536 and gz == 1, (c, w)
            assert gx * gy * 64 * 64 >= c["T"] * width, (c, w)


if __name__ == "__main__":
    _child(sys.argv[1], sys.argv[2], json.loads(sys.argv[3]))
