"""What the library launches for a call, seen from the host: its own host code runs against a stand-in for the HIP runtime
(hip_host_stub.cpp) that records every launch and refuses what the runtime would refuse.  No GPU is used."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys, threading
sys.path.insert(0, {root!r})
stub = ctypes.CDLL({stub!r}, mode=ctypes.RTLD_GLOBAL)
stub.stub_records.restype = ctypes.c_char_p
import paper_1706_09453_amd as bnn
A, B, C, D, E = (0x1000000000 * i for i in range(1, 6))    # made-up device addresses, far apart
def launches():
    out = []
    for line in stub.stub_records().decode().splitlines():
        w = line.split()
        out.append(dict(kernel=w[0], grid=[int(v) for v in w[1:4]], block=int(w[4]), lds=int(w[5]), device=int(w[6]), wrong=w[7:]))
    stub.stub_clear()
    return out
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    """host(code): runs `code` in a process of its own, where launches() lists what was launched; returns its `result`."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    stub = str(tmp_path_factory.mktemp("stub") / "libhip_host_stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread", "-o", stub, os.path.join(HERE, "hip_host_stub.cpp")], check=True)

    def run(code):
        src = PRELUDE.format(root=ROOT, stub=stub) + code + "\nimport json; print('RESULT ' + json.dumps(result))\n"
        res = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=120)
        assert res.returncode == 0, res.stderr[-2000:]
        return json.loads(res.stdout.split("RESULT ", 1)[1])

    return run


def test_norm_inside_the_workspace_is_written_before_the_gradient_is_scaled(host):
    """norm_out may lie in the 2048 bytes of partial sums: the launch that scales must then not be the one that stores the
    norm, since its other workgroups still read the sums."""
    got = host("""
result = []
for norm in (B, B + 4, B + 2044, B + 2048, C):
    bnn.bnn_grad_norm_clip(A, 1 << 20, 15.0, B, norm)
    result.append([l["kernel"] for l in launches()])
""")
    for kernels in got[:3]:
        assert len(kernels) == 3 and "sumsq_partial" in kernels[0] and "sumsq_final" in kernels[1] and "scale_if_above" in kernels[2], kernels
    for kernels in got[3:]:
        assert len(kernels) == 2 and "sumsq_partial" in kernels[0] and "scale_if_above" in kernels[1], kernels


FORWARD = """
def forward(M, dims=(440, 2048), acts=(bnn.BNN_ACT_SIGN,), real=(), out=D):
    d, binary = [], 0
    for l, a in enumerate(acts):
        d.append(dict(K=dims[l], N=dims[l + 1], act=a, word_bits=32, x_is_binary=binary, w_is_real=l in real, Wp=B + l * 0x10000000,
                      scale=0 if l in real else C, bias=C))
        binary = int(a == bnn.BNN_ACT_SIGN)
    arr = bnn.make_layer_array(d)
    bnn.bnn_forward(arr, len(d), A, M, out, E, bnn.bnn_forward_workspace_bytes(arr, len(d), M), 0)
"""


def test_lds_is_allowed_on_every_device(host):
    """Dynamic LDS above 64 KiB is allowed per device: a second device is asked too, whichever kernel it is."""
    got = host(FORWARD + """
Z, H, S, G = bnn.BNN_ACT_LOGSOFTMAX, bnn.BNN_ACT_HARDTANH, bnn.BNN_ACT_SIGN, bnn.BNN_ACT_SIGMOID
for dev in (0, 1, 70, 6):
    stub.stub_set_device(dev)
    for M in (100, 333, 4096):
        forward(M)                                                   # first layer, Sign
        forward(M, (440, 2048, 2048, 3400), (G, S, Z))               # real inputs further on, real outputs
        forward(M, (440, 2048, 3400), (H, Z))
        forward(M, (440, 2048, 3400), (G, Z), real=(0, 1))           # real weights
    for opt, v in ((bnn.BNN_OPT_REALX_SIGN_MFMA, 2), (bnn.BNN_OPT_REALX_I8_LOGSOFTMAX, 2), (bnn.BNN_OPT_REALW_SPLIT_LOGSOFTMAX, 2)):
        bnn.bnn_set_option(opt, v)
        forward(333, (440, 2048, 2048, 3400), (G, S, Z))
        forward(333, (440, 2048, 3400), (H, Z))
        forward(333, (440, 2048, 3400), (G, Z), real=(0, 1))
        bnn.bnn_set_option(opt, 1)
result = launches()
""")
    assert {l["device"] for l in got if l["lds"] > 65536} == {0, 1, 70, 6}
    assert not [l for l in got if l["wrong"]]


def test_lds_of_two_batch_sizes_at_once(host):
    """The first layer's LDS depends on the batch: two threads that ask for it at the same time both get what they need."""
    got = host(FORWARD + """
first = threading.Thread(target=forward, args=(4096,))    # all 2048 outputs in one workgroup: the most LDS
stub.stub_hold_next_grant()
first.start()
import time
time.sleep(0.2)
forward(333, out=D + 0x10000000)
first.join()
forward(4096)
result = launches()
""")
    assert len(got) == 3 and len({l["lds"] for l in got}) == 2 and min(l["lds"] for l in got) > 65536
    assert not [l for l in got if l["wrong"]]


def test_bias_grad_grids(host):
    """The sums of a wide matrix take one wave per 64 columns, and every width up to 2^30 columns has a grid that the
    runtime accepts."""
    got = host("""
bnn.bnn_bias_grad(A, 4096, 12288, D)
for M, N in ((1, 12289), (64, 20000), (1, 1 << 28), (1, (1 << 30) - 1), (1, 1 << 30)):
    bnn.bnn_bias_grad(A, M, N, D)
result = launches()
""")
    assert "colsum_kernel" in got[0]["kernel"] and got[0]["grid"][0] == 768
    for l in got[1:]:
        assert "colsum_wave_kernel" in l["kernel"] and l["block"] == 64 and not l["wrong"]
    assert [l["grid"][0] for l in got[1:3]] == [193, 313]


def test_softmax_gradient_spreads_elements_over_the_chip(host):
    """Few classes or few frames: as many threads as there are elements (or groups of four), not a workgroup per frame."""
    got = host("""
for M, N, off in ((50000, 4, 0), (1, 100000, 0), (16, 3400, 0), (50000, 10, 0), (1, 100000, 4), (4096, 3400, 0)):
    bnn.bnn_softmax_xent_grad(A + off, B, M, N, C)
result = launches()
""")
    assert [l["grid"][0] for l in got] == [196, 98, 54, 1954, 391, 4096] and all(l["block"] == 256 for l in got)


def test_packing_takes_no_more_per_wave_than_a_row_holds(host):
    """64, 128, 256 or 512 numbers of a row per wave: short rows do not load theirs several times over."""
    got = host("""
for K in (1, 64, 65, 128, 129, 256, 257, 2048):
    bnn.bnn_pack_activations(A, 4096, K, 32, D)
result = launches()
""")
    ballots = [int(l["kernel"].split("pack_sign_kernelILi")[1].split("E")[0]) for l in got]
    assert ballots == [1, 1, 2, 2, 4, 4, 8, 8]
    assert [l["grid"][0] for l in got] == [1024] * 7 + [4096]


def _chain_tile(kernel):
    """256x128x32 and so on from the kernel's template arguments (FM, FN, WR, KC, ACT, WREAL, VEC, SKIP)."""
    if "f32_chain_kernel" not in kernel:
        return "valu" if "valu" in kernel else kernel
    args = kernel.split("f32_chain_kernelI")[1].split("E")
    fm, fn, wr, kc = (int(a[2:]) for a in args[:4])
    real, vec, skip = (a[2:] == "1" for a in args[5:8])
    return f"{16 * fm * wr}x{64 * fn // wr}x{kc}" + ("+" if skip else "") + ("" if vec else ":1")


def test_every_tile_of_the_ascending_sums_is_among_the_tested_sizes(host):
    """The sizes the GPU tests run take the tiles they are listed for, and no tile the dispatch picks anywhere in its range is
    missing among them."""
    from chain_sizes import CHAIN_TILES
    got = host("""
sizes = %r
result = []
for M, K, N in sizes:
    for real in (0, 1):
        if real:
            bnn.bnn_layer_realw(A, B, C, M, K, N, bnn.BNN_ACT_LINEAR, 32, D)
        else:
            bnn.bnn_layer_binw_realx(A, B, C, C, M, K, N, bnn.BNN_ACT_LINEAR, 32, D)
        result.append(launches())
seen = set()
for M in (1, 16, 17, 64, 65, 100, 200, 333, 512, 777, 1000, 1500, 2048, 3000, 4096, 16384):
    for K in (1, 4, 8, 16, 24, 31, 32, 33, 36, 48, 60, 64, 68, 100, 143, 429, 440, 1024, 2047, 2048):
        for N in (1, 64, 100, 512, 1000, 1024, 2048, 3400, 4096, 30000):
            bnn.bnn_layer_realw(A, B, C, M, K, N, bnn.BNN_ACT_LINEAR, 32, D)
            bnn.bnn_layer_binw_realx(A, B, C, C, M, K, N, bnn.BNN_ACT_LINEAR, 32, D)
for l in launches():
    assert not l["wrong"], l
    seen.add(l["kernel"])
result = [result, sorted(seen)]
""" % [s for s, _, _ in CHAIN_TILES])
    per_size, seen = got
    tested = set()
    for i, (size, bits, real) in enumerate(CHAIN_TILES):
        for launched, want in ((per_size[2 * i], bits), (per_size[2 * i + 1], real)):
            assert len(launched) == 1 and _chain_tile(launched[0]["kernel"]) == want, (size, launched)
            tested.add(launched[0]["kernel"])
    chains = [k for k in seen if "f32_chain_kernel" in k]
    assert len(chains) >= 16 and not set(chains) - tested


def test_binary_layers_take_the_kernel_their_size_wants(host):
    """Exceptions to the line at 256 tiles of 32 x 128: short output layers hand int16 over, integer outputs of few frames
    stay on 64-row tiles; and rows whose pad bits complete their 512-bit pieces are read 16 bytes at a time."""
    got = host("""
Z, R, S = bnn.BNN_ACT_LOGSOFTMAX, bnn.BNN_ACT_RAW_I32, bnn.BNN_ACT_SIGN
result = []
for M, K, N, act in ((1024, 512, 1000, Z), (512, 512, 64, Z), (511, 512, 64, Z), (1000, 1024, 1000, Z), (512, 1024, 512, Z), (1000, 2048, 512, Z),
                     (1000, 64, 3400, R), (1000, 512, 3400, R), (1024, 64, 3400, R), (1000, 64, 3400, S),
                     (100, 1000, 512, S), (100, 960, 512, S), (100, 993, 512, S)):
    bnn.bnn_layer_binw_binx(A, B, C, C, M, K, N, act, 32, D)
    result.append(launches()[0]["kernel"])
""")
    small, large = "binx_mfma_kernel", "binx_mfma32_kernel"
    assert [large if large in k else small for k in got] == [large, large, small, large, small, small, small, large, large, large, small, small, small]
    assert "Li4ELi4ELi0E" in got[6]                                   # 64-row tiles
    assert ["Lb1ELb0E" in k for k in got[10:]] == [True, False, True]  # ALIGNED


def test_binary_layers_of_one_stage_take_64_row_tiles(host):
    """K = 512 is one stage of the kernel that fetches through LDS: 64-row tiles, unless only the 128-row ones are done in one round
    of workgroups, or the cooperative log-Softmax, which has 128-row tiles only, is asked for."""
    got = host("""
Z, S = bnn.BNN_ACT_LOGSOFTMAX, bnn.BNN_ACT_SIGN
result = []
for coop in (0, 1):
    bnn.bnn_set_option(bnn.BNN_OPT_COOPERATIVE, coop)
    for M, K, N, act in ((16384, 512, 4096, S), (1798, 512, 6816, S), (16384, 1024, 4096, S), (1500, 1024, 2048, S), (4096, 512, 2048, Z), (4096, 1024, 2048, Z)):
        bnn.bnn_layer_binw_binx(A, B, C, C, M, K, N, act, 32, D)
        l = launches()[0]
        result.append([l["kernel"].split("binx_mfma32_kernelILi")[1][0], l["wrong"]])
""")
    assert [w for w, _ in got] == ["2", "4", "4", "2", "2", "4", "2", "4", "4", "2", "4", "4"]
    assert not [w for _, w in got if w]


def test_softmax_layer_with_real_weights_tiles_and_long_rows(host):
    """Which tile of the bf16-piece product a layer takes, by rounds of workgroups; and rows whose offsets in a tile would not fit 32
    bits take the instantiation with 64-bit addresses, on every size the entry point accepts."""
    got = host(FORWARD + """
result = []
for M, K, N in ((128, 64, 1), (600, 2048, 3400), (2049, 289, 3329), (4096, 2048, 3400), (4096, 2048, 1000), (2600, 2048, 3400),
                (1 << 12, (1 << 22) - 32, 1 << 13), (128, (1 << 22) - 31, 7), (4096, 1 << 22, 8192), (300, 1 << 23, 130), (128, 1 << 24, 7), (128, 1 << 30, 1)):
    forward(M, (K, N), (bnn.BNN_ACT_LOGSOFTMAX,), real=(0,), out=0x700000000000)
    l = [l for l in launches() if "realw_bf16x3_kernel" in l["kernel"]][0]
    t = l["kernel"].split("realw_bf16x3_kernelI")[1].split("E")
    result.append([t[0][2:] + "x" + t[1][2:] + ("" if t[2] == "Lb0" else " long"), l["grid"][:2], l["wrong"]])
""")
    assert [k for k, _, _ in got] == ["2x2", "2x2", "4x2", "4x2", "2x2", "2x2", "4x2", "2x2 long", "2x2 long", "2x2 long", "2x2 long", "2x2 long"]
    assert got[1][1] == [5, 27] and got[2][1] == [9, 27] and got[9][1] == [3, 2]
    assert not [w for _, _, w in got if w]


def test_static_forward_is_not_charged_for_memory_no_kernel_uses(host):
    """A hidden layer with real weights: what bnn_forward only reserves for it does not keep the tiled products out of the
    fixed array.  The size a caller provides stays what it was."""
    got = host(FORWARD + """
H, Z = bnn.BNN_ACT_HARDTANH, bnn.BNN_ACT_LOGSOFTMAX
dims, acts = (300, 2048, 2048, 1000), (H, H, Z)
forward(512, dims, acts, real=(1,))
want = [l["kernel"] for l in launches()]
d = [dict(K=dims[l], N=dims[l + 1], act=acts[l], word_bits=32, x_is_binary=0, w_is_real=l == 1, Wp=B + l * 0x10000000,
          scale=0 if l == 1 else C, bias=C) for l in range(3)]
arr = bnn.make_layer_array(d)
bnn.bnn_forward_static(arr, 3, A, 512, D, 0)
result = [want, [l["kernel"] for l in launches()], bnn.bnn_forward_workspace_bytes(arr, 3, 512)]
""")
    assert got[0] == got[1] and any("realx_i8_gemm" in k for k in got[0])
    assert got[2] == 2 * 512 * 2048 * 4 + 2048 * 2048 * 4


def test_int8_product_tiles_by_rounds_of_workgroups(host):
    """64 x 128 tiles (two workgroups per CU) where their rounds cost less than those of 128 x 256 tiles."""
    got = host("""
result = []
def call(M, N, K):
    n = bnn.bnn_layer_binw_realx_i8_workspace_bytes(M, K, N)
    bnn.bnn_layer_binw_realx_i8(A, B, 0, 0, M, K, N, 32, 0x800000000000, 0x700000000000, n, 0)
    l = [l for l in launches() if "realx_i8_gemm_kernel" in l["kernel"]][0]
    result.append([l["kernel"], l["grid"], l["wrong"]])
for M, N in ((1, 1), (600, 3400), (2048, 2048), (2600, 2048), (4096, 2048), (2049, 2049), (4096, 3400), (1 << 25, 1)):
    call(M, N, 64)
""")
    small = ["Li1ELi2E" in k for k, _, _ in got]
    assert small == [True, True, True, False, False, False, False, True]
    assert got[1][1][:2] == [10, 27] and got[4][1][:2] == [32, 8]
    assert not [w for _, _, w in got if w]


def test_a_run_of_binary_layers_follows_a_launch_that_clears_its_marks(host):
    """Whatever another thread does to the options while a forward pass chooses its kernels: a run in one launch comes only behind a
    kernel that clears what the run trusts (such kernels take a Clear), never behind the slab kernel, which does not."""
    runs, uncleared = host("""
G, S = bnn.BNN_ACT_SIGMOID, bnn.BNN_ACT_SIGN
def network(N):
    dims, acts = (440, 600) + (N,) * 6, (G,) + (S,) * 6
    return bnn.make_layer_array([dict(K=dims[l], N=dims[l + 1], act=acts[l], word_bits=32, x_is_binary=int(l > 1), w_is_real=0,
                                      Wp=B + l * 0x10000000, scale=C, bias=C) for l in range(7)])
stub.stub_turn.argtypes = [ctypes.c_void_p] + [ctypes.c_int] * 3
set_option = ctypes.cast(bnn.binding._lib.bnn_set_option, ctypes.c_void_p)
runs = uncleared = 0
for M, N in ((64, 64), (200, 512)):
    for option, one, other in ((bnn.BNN_OPT_REALX_SIGN_MFMA, 2, 1), (bnn.BNN_OPT_STREAM_MAX_FRAMES, 0, 64)):
        arr = network(N)
        size = bnn.bnn_forward_workspace_bytes(arr, 7, M)
        stub.stub_turn(set_option, option, one, other)
        for _ in range(1000):
            bnn.bnn_forward(arr, 7, A, M, D, E, size, 0)
            kernels = [l["kernel"] for l in launches()]
            for before, k in zip(kernels, kernels[1:]):
                if "few_chain_kernel" in k or "hidden_run_kernel" in k:
                    runs += 1
                    uncleared += "Clear" not in before
        stub.stub_turn_end()
result = [runs, uncleared]
""")
    assert runs > 100 and uncleared == 0


def test_which_binary_layers_share_a_launch(host):
    """Runs of a few frames and of mid-size batches, on both sides of each line."""
    got = host(FORWARD + """
S, Z = bnn.BNN_ACT_SIGN, bnn.BNN_ACT_LOGSOFTMAX
result = []
for M, widths in ((1, (512, 512)), (1, (512, 512, 512)), (1, (520, 512)), (64, (2048, 2048, 2048)), (64, (2049, 2049, 2049)), (17, (4096, 2048, 2048)),
                  (4096, (512, 512)), (4097, (512, 512)), (1024, (1024, 1024)), (1025, (1024, 1024)), (512, (1536, 1536)), (513, (1536, 1536)),
                  (128, (2048, 2048)), (129, (2048, 2048)), (65, (1000, 1000)), (65, (512, 1024)),
                  (17, (1024, 1024, 1024)), (17, (1025, 1025, 1025))):
    for last in (None, 100):
        dims = (40, widths[0]) + widths + ((last,) if last else ())
        forward(M, dims, (S,) * (len(dims) - 1 - bool(last)) + ((Z,) if last else ()))
        k = [l for l in launches() if "few_chain" in l["kernel"] or "hidden_run" in l["kernel"]]
        result.append([("few" if "few_chain" in l["kernel"] else "mid") + str(l["grid"][0]) for l in k])
""")
    few, pulling, mid = ["few256"], ["few512"], ["mid256"]
    # (without, with an output layer): two binary layers of whole pieces are a run only with the log-Softmax behind them; 512 workgroups: half of them pull
    want = [[], few, few, few, few, few, few, few, [], [], [], [],
            mid, mid, [], [], mid, mid, [], [], mid, mid, [], [], mid, mid, [], [], [], [], [], [],
            pulling, pulling, few, few]
    assert got == want, [(i, g, w) for i, (g, w) in enumerate(zip(got, want)) if g != w]


def test_workspace_without_the_scratch_of_runs(host):
    """The size of that scratch is what bnn.h says; without it a launch per layer, with less BNN_EWORKSPACE."""
    got = host("""
S, Z = bnn.BNN_ACT_SIGN, bnn.BNN_ACT_LOGSOFTMAX
up = lambda v: (v + 255) // 256 * 256
result = []
for M, dims, last, scratch in ((1, (40, 512, 512, 1001), Z, up(8 * (16 + 128)) + up(1002 * 4)), (50, (40, 1000, 90, 1024, 70), S, up(8 * 50 * 2 * 32)),
                               (33, (40, 2048, 2048, 7, 4096), Z, up(8 * 33 * (2 * 64 + 128)) + up(33 * 4096 * 4)),
                               (333, (40, 1024, 1024, 1024, 70), Z, 2 * 4096 + up(333 * 128)), (130, (600, 512, 512, 512, 512), S, 3 * 4096 + 2 * up(130 * 64))):
    n = len(dims) - 1
    arr = bnn.make_layer_array([dict(K=dims[l], N=dims[l + 1], act=S if l < n - 1 else last, word_bits=32, x_is_binary=int(l > 0), w_is_real=0,
                                     Wp=B + l * 0x10000000, scale=C, bias=C) for l in range(n)])
    total = bnn.bnn_forward_workspace_bytes(arr, n, M)
    row = []
    for size in (total, total - 1, total - scratch, total - scratch - 1):
        try:
            bnn.bnn_forward(arr, n, A, M, D, E, size, 0)
            row.append(sum("few_chain" in l["kernel"] or "hidden_run" in l["kernel"] for l in launches()))
        except bnn.BnnError as e:
            row.append(str(e))
    result.append(row)
""")
    for row in got:
        assert row[:3] == [1, 0, 0] and "workspace" in str(row[3]).lower(), row


def test_no_run_writes_over_weights_it_still_reads(host):
    """The output may lie where a layer before the last one keeps its weights: then every layer takes a launch of its own."""
    got = host(FORWARD + """
S, Z = bnn.BNN_ACT_SIGN, bnn.BNN_ACT_LOGSOFTMAX
result = []
for M, dims, acts in ((8, (40, 512, 512, 512, 70), (S, S, S, Z)), (200, (40, 512, 512, 512, 512), (S, S, S, S))):
    for out in (D, B + 0x10000000 + 512 * 64 - 16, B + 0x10000000 + 512 * 64):   # (the first layer of the run: 32 KB of weights)
        forward(M, dims, acts, out=out)
        result.append(sum("few_chain" in l["kernel"] or "hidden_run" in l["kernel"] for l in launches()))
""")
    assert got == [1, 0, 1, 1, 0, 1]
