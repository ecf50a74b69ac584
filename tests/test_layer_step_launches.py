"""What moe_layer_step launches, recorded on the host by a stand-in for the HIP runtime (no GPU needed).

A child process loads a few C functions in place of the runtime's (kernel registration and launch) ahead of
the library, calls it with made-up device addresses, which only kernels would follow, and prints the names of
the kernels in launch order.
"""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = textwrap.dedent('''
    #include <stddef.h>
    #include <stdint.h>
    #include <stdio.h>
    #include <string.h>
    typedef struct { uint32_t x, y, z; } dim3;
    static struct { const void* fn; const char* name; } kernels[1024];
    static int n_kernels;
    static struct { dim3 grid, block; size_t shared; void* stream; } config;
    static void* module;
    static char log_[1 << 16];
    static void (*hook)(int);
    static int n_launches;
    static void** last_args;
    void** __hipRegisterFatBinary(const void* data) { (void)data; return &module; }
    void __hipUnregisterFatBinary(void** m) { (void)m; }
    void __hipRegisterFunction(void** m, const void* fn, char* device, const char* name, unsigned limit, void* tid,
                               void* bid, dim3* block, dim3* grid, int* size) {
        (void)m; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)size;
        kernels[n_kernels].fn = fn;
        kernels[n_kernels++].name = name;
    }
    void __hipRegisterVar(void** m, void* v, char* a, char* b, int c, size_t d, int e, int f) {
        (void)m; (void)v; (void)a; (void)b; (void)c; (void)d; (void)e; (void)f;
    }
    int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void* stream) {
        config.grid = grid; config.block = block; config.shared = shared; config.stream = stream;
        return 0;
    }
    int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, void** stream) {
        *grid = config.grid; *block = config.block; *shared = config.shared; *stream = config.stream;
        return 0;
    }
    int hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t shared, void* stream) {
        (void)block; (void)shared; (void)stream;
        for (int i = 0; i < n_kernels; ++i)
            if (kernels[i].fn == fn) {
                const size_t at = strlen(log_);
                snprintf(log_ + at, sizeof(log_) - at, "%s %u\\n", kernels[i].name, grid.x);
            }
        last_args = args;
        if (hook) hook(++n_launches);
        return 0;
    }
    int hipGetLastError(void) { return 0; }
    int hipEventRecord(void* e, void* stream) { (void)e; (void)stream; return 0; }
    int hipGetDevice(int* d) { *d = 0; return 0; }
    int hipFuncSetAttribute(const void* fn, int a, int v) { (void)fn; (void)a; (void)v; return 0; }
    int hipGetDevicePropertiesR0600(void* p, int d) { (void)p; (void)d; return 1; }
    int int_argument(int i) { return *(int*)last_args[i]; }   /* of the launch under way */
    const char* launches(void) { return log_; }
    void start(void (*h)(int)) { log_[0] = 0; n_launches = 0; hook = h; }
''')

CHILD = textwrap.dedent('''
    import ctypes, struct, sys
    rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    lib = ctypes.CDLL(sys.argv[2])
    c_int, c_i64, c_sz = ctypes.c_int, ctypes.c_int64, ctypes.c_size_t
    rt.launches.restype = ctypes.c_char_p
    lib.moe_grouped_ffn_workspace_bytes.restype = lib.moe_permute_workspace_bytes.restype = c_sz
    lib.moe_grouped_ffn_workspace_bytes.argtypes = [c_i64] + [c_int] * 4
    lib.moe_layer_step.argtypes = [ctypes.c_char_p, ctypes.c_void_p]
    HOOK = ctypes.CFUNCTYPE(None, c_int)
    rt.start.argtypes = [HOOK]
    POINTERS = ("logits x hist_pred pred_idx packed topk_idx topk_w hist hist_plan slot_expert slot_quota rank_load_pred "
                "n_iters seg_offsets row_of_assign assign_of_row x_perm rank_load y_perm out").split()
    MODE, DTYPE, T, D, FFN, E, K, G, S, CMAX, RELU, GATE = range(12)

    def step(ints, hook=None, ws=(0, 0), **pointers):
        """(return code, launches) of a step; pointers far apart unless given, ws: bytes missing from the workspaces"""
        p = {n: (i + 1) << 40 for i, n in enumerate(POINTERS)}
        p.update(pointers)
        A = max(ints[T], 0) * max(ints[K], 1)
        perm = lib.moe_permute_workspace_bytes(ints[T], ints[E], ints[K], ints[G], ints[S]) - ws[0]
        ffn = lib.moe_grouped_ffn_workspace_bytes(A, ints[D], ints[FFN], ints[G] * ints[S] & 0x7fffffff, ints[DTYPE]) - ws[1]
        args = struct.pack("@12i24Q", *ints, *[p[n] for n in POINTERS], p.get("ws_perm", 21 << 40), max(perm, 0),
                           p.get("ws_ffn", 22 << 40), max(ffn, 0))
        keep = HOOK(hook) if hook else HOOK()
        rt.start(keep)
        rc = lib.moe_layer_step(args, None)
        got = rt.launches().decode()
        return rc, [l.split()[0] for l in got.splitlines()]
''')


@pytest.fixture(scope="module")
def child(tmp_path_factory):
    """Runs a script behind CHILD; its output."""
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no C compiler")
    from paper_2506_07366_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2506_07366_amd.build import build
        build(verbose=False)
    tmp = tmp_path_factory.mktemp("runtime")
    (tmp / "rt.c").write_text(RUNTIME)
    rt = str(tmp / "rt.so")
    subprocess.run([cc, "-shared", "-fPIC", "-o", rt, str(tmp / "rt.c")], check=True)

    def run(script):
        path = tmp / "child.py"
        path.write_text(CHILD + textwrap.dedent(script))
        r = subprocess.run([sys.executable, str(path), rt, binding.LIB_PATH], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, f"{r.stdout}\n{r.stderr}"
        return r.stdout

    return run


def test_options_are_read_once_per_step(child):
    """An option that another thread sets while a step is under way is for the next one: the products are those
    whose tables the permutation has built."""
    out = child('''
        TILE1, TILE2, SPLIT, GROUP_N, STREAM = range(5)
        for ints in ([1, 1, 16, 4096, 1024, 8, 2, 8, 3, 8, 0, 0],       # streams: tables by the permutation
                     [1, 1, 1500, 512, 2048, 8, 2, 8, 3, 8, 0, 0]):     # tiles, closing ones split
            want = step(ints)
            assert want[0] == 0, want
            for option, value in ((STREAM, 0), (STREAM, 1), (STREAM, 2), (TILE1, 1), (TILE2, 2), (SPLIT, 0), (SPLIT, 1)):
                for after in range(1, len(want[1])):
                    hook = lambda n: n == after and lib.moe_grouped_ffn_set_option(option, value)
                    got = step(ints, hook)
                    lib.moe_grouped_ffn_set_option(option, -1)
                    assert got == want, (option, value, after, got, want)
            print(len(want[1]), "launches")
    ''')
    assert out.count("launches") == 2


@pytest.mark.parametrize("option", [1, 7, 8, 9, 2**16, 2**31 - 1])
def test_n_tiles_walked_together_are_tiles_that_exist(child, option):
    """The tile kernel multiplies the option by its M-tiles: it gets no more than there are N-tiles."""
    out = child(f"""
        N, GROUP = 9, 11                      # arguments of grouped_gemm_tile_kernel
        def look(n):
            if "grouped_gemm_tile" in rt.launches().decode().splitlines()[-1]:
                print("tile", rt.int_argument(N), rt.int_argument(GROUP))
        assert lib.moe_grouped_ffn_set_option(3, {option}) == 0
        assert step([1, 1, 1500, 512, 1024, 8, 2, 8, 3, 8, 0, 0], look)[0] == 0
    """)
    seen = [tuple(map(int, line.split()[1:])) for line in out.splitlines() if line.startswith("tile")]
    assert seen == [(2048, min(option, 8)), (512, min(option, 2))]


def test_own_outputs_as_prediction_come_in_the_order_of_the_single_calls(child):
    """ids or counts that the step itself writes: routing, histogram (of the predicted ids too), plan, permutation, each a
    launch of its own.  A prediction next to them shares the launches as any other does."""
    out = child("""
        def kinds(mode, t, e, g, s, **pointers):
            rc, names = step([mode, 1, t, 64, 64, e, 2, g, s, 8, 0, 0], **pointers)
            assert rc == 0
            return [next(w for w in ("route_plan", "route", "hist", "plan", "perm", "other") if w in n or w == "other")
                    for n in names]
        TOPK, WEIGHT, HIST = [(POINTERS.index(n) + 1) << 40 for n in ("topk_idx", "topk_w", "hist")]
        for shape in ((64, 16, 4, 5), (3000, 16, 4, 5), (100, 300, 32, 10)):
            ids, counts = 2 * shape[0] * 4, shape[1] * 4
            for at in (TOPK, TOPK - ids + 4, TOPK + ids - 4, WEIGHT, HIST + counts - 4):
                got = kinds(2, *shape, pred_idx=at)
                assert got[:5] == ["route", "hist", "hist", "plan", "perm"], (shape, at, got)
            for at in (HIST, HIST - counts + 4, HIST + counts - 4, TOPK, WEIGHT + ids - 4):
                got = kinds(1, *shape, hist_pred=at)
                assert got[:4] == ["route", "hist", "plan", "perm"], (shape, at, got)
            for mode, beside in ((2, dict(pred_idx=TOPK - ids)), (2, dict(pred_idx=TOPK + ids)), (1, dict(hist_pred=HIST + counts)),
                                 (1, dict(pred_idx=TOPK)), (2, dict(hist_pred=HIST)), (0, dict(pred_idx=TOPK, hist_pred=HIST))):
                assert kinds(mode, *shape, **beside) == kinds(mode, *shape), (shape, mode, beside)
            print("shape", kinds(2, *shape))
    """)
    assert out.count("shape") == 3


def test_arguments_are_checked_before_the_first_launch(child):
    """What the single calls refuse is refused, with their codes, and nothing has been launched by then."""
    child("""
        INVALID, UNSUPPORTED, TOO_SMALL = -1, -2, -3
        good = [1, 1, 16, 64, 64, 8, 2, 8, 2, 8, 0, 0]
        assert step(good)[0] == 0 and len(step(good)[1]) > 3
        def refused(code, changes={}, **kw):
            ints = list(good)
            for i, v in changes.items():
                ints[i] = v
            got = step(ints, **kw)
            assert got == (code, []), (changes, kw, got)
        for field, value in ((MODE, -1), (MODE, 3), (DTYPE, 2), (T, -1), (D, 0), (FFN, 0), (E, 0), (K, 0), (K, 9), (G, 0), (S, 0),
                             (CMAX, 0), (G, 2)):                       # (two ranks of two slots do not hold 8 experts)
            refused(INVALID, {field: value})
        for changes in ({E: 1025, G: 256, S: 8}, {E: 17, K: 17, G: 16}, {G: 257}, {S: 17}, {G: 256, S: 9}, {D: 4}, {D: 72},
                        {D: 63, DTYPE: 0}, {FFN: 66, DTYPE: 0}, {FFN: (1 << 22) + 1}, {D: 1 << 23}, {T: 1 << 30},
                        {T: 1 << 25}, {T: 1 << 28, E: 9, K: 1, G: 9, D: 4, FFN: 4, DTYPE: 0}):
            refused(UNSUPPORTED, changes)
        for name in POINTERS:
            if name in ("pred_idx", "hist_plan", "x_perm"):
                continue
            refused(INVALID, {}, **{name: 0})
        for name in ("ws_perm", "ws_ffn"):
            refused(INVALID, {}, **{name: 0})
        refused(INVALID, {MODE: 2}, pred_idx=0)
        refused(INVALID, {MODE: 2}, hist_plan=0)
        refused(UNSUPPORTED, {RELU: 1}, x_perm=0)
        refused(TOO_SMALL, {}, ws=(1, 0))
        refused(TOO_SMALL, {}, ws=(0, 1))
        assert step([0, 1, 0] + good[3:]) == (0, [])                   # no tokens: nothing to do
        for ints, kw in (([0] + good[1:], dict(hist_pred=0, pred_idx=0, hist_plan=0)), (good, dict(pred_idx=0, hist_plan=0)),
                         ([2] + good[1:], dict(hist_pred=0)), (good, dict(x_perm=0)), (good[:11] + [1], dict(x_perm=0))):
            assert step(ints, **kw)[0] == 0, (ints, kw)                # what a mode does not read may be missing
    """)


def test_products_share_a_launch_only_where_hidden_rows_are_whole_cache_lines(child):
    """The hidden rows lie at the start of the FFN's scratch, of which the ABI asks 16 bytes of alignment: where a row shares a
    128-byte line with the next one, a launch that reads finished rows beside unfinished ones is not to be had."""
    out = child("""
        FFN_WS = 22 << 40
        for at in (0, 16, 32, 48, 64, 80, 96, 112, 128, 144, 192, 256, 4096 + 64):
            for relu, x_perm in ((0, 17 << 40), (1, 17 << 40), (0, 0)):
                rc, names = step([1, 1, 3000, 1024, 3008 if relu else 2048, 8, 2, 4, 3, 8, relu, 0], ws_ffn=FFN_WS + at, x_perm=x_perm)
                assert rc == 0
                products = [n for n in names if "grouped_" in n]
                assert len(products) == (1 if at % 128 == 0 else 2), (at, relu, products)
                assert ("grouped_ffn_tiles" in products[0]) == (at % 128 == 0), (at, products)
                print("step")
    """)
    assert out.count("step") == 39


def test_outputs_in_the_logits_are_written_once_these_are_read(child):
    """No workgroup clears the histogram or writes the plan beside others that still route: where one of these outputs lies in the
    logits, a later launch does."""
    out = child("""
        LOGITS = (POINTERS.index("logits") + 1) << 40
        def kinds(mode, t, e, g, s, **pointers):
            rc, names = step([mode, 1, t, 64, 64, e, 2, g, s, 8, 0, 0], **pointers)
            assert rc == 0
            return [next(w for w in ("route_plan", "route", "hist", "plan", "perm", "other") if w in n or w == "other") for n in names]
        for shape in ((64, 16, 4, 5), (3000, 16, 4, 5), (20000, 16, 4, 5)):   # one workgroup permutes; several; ids counted ahead
            t, e, g, s = shape
            size = dict(hist=4 * e, hist_plan=4 * e, slot_expert=4 * g * s, slot_quota=4 * g * s, rank_load_pred=4 * g, n_iters=4)
            for mode in (0, 1, 2):
                beside = kinds(mode, *shape)
                for name, n in size.items():
                    for at in (LOGITS + 4 * t * e, LOGITS - n):
                        assert kinds(mode, *shape, **{name: at}) == beside, (shape, mode, name)
                    for at in (LOGITS, LOGITS + 4 * t * e - 4, LOGITS + 4 - n):
                        got = kinds(mode, *shape, **{name: at})
                        if name == "hist" and t > 1000:                  # the launch after the routing's and the plan's makes it whole
                            assert got[:3] == {0: ["route", "hist", "plan"], 1: ["route_plan", "hist", "perm"],
                                               2: ["hist", "route_plan", "hist"] if t > 10000 else ["route_plan", "hist", "perm"]}[mode]
                        elif name == "hist" or mode == 0 or (name == "hist_plan" and mode != 2):
                            assert got == beside, (shape, mode, name, got)   # not written yet, or not at all
                        else:
                            assert got[0] == "route" and "route_plan" not in got, (shape, mode, name, got)
            print("shape")
    """)
    assert out.count("shape") == 3


@pytest.mark.parametrize("T,d,ffn,E,k,relu,both", [
    (1408, 1024, 2048, 8, 2, 0, False), (1409, 1024, 2048, 8, 2, 0, True),       # a round of 256 tiles
    (13824, 1024, 2048, 8, 2, 0, True), (13825, 1024, 2048, 8, 2, 0, False),     # seven
    (3000, 704, 2048, 8, 2, 0, False), (3000, 768, 2048, 8, 2, 0, True),         # 12 k-tiles in the first product
    (3000, 1024, 4032, 8, 2, 0, True), (3000, 1024, 4033, 8, 2, 0, False),       # 63 in the second
    (3000, 1024, 4032, 8, 2, 1, True), (3000, 1024, 4096, 8, 2, 1, False),
    (384, 4096, 14336, 8, 2, 0, False), (1001, 4096, 14336, 8, 2, 0, False), (1400, 4096, 14336, 8, 2, 0, False),
])
def test_products_share_a_launch_within_the_rule(child, T, d, ffn, E, k, relu, both):
    out = child(f"""
        rc, names = step([1, 1, {T}, {d}, {ffn}, {E}, {k}, 8, 2, 8, {relu}, 0])
        assert rc == 0
        print(["tiles" if "grouped_gemm_tile" in n else "both" for n in names if "grouped_" in n])
    """)
    assert out.strip() == str(["both"] if both else ["tiles", "tiles"]), out


def test_a_call_with_events_is_a_launch_per_product(child):
    """... and the next one, without, runs both in one again."""
    out = child("""
        ints = [1, 1, 3000, 1024, 2048, 8, 2, 4, 3, 8, 0, 0]
        events = (ctypes.c_void_p * 4)(1, 2, 3, 4)
        for armed in (False, True, False):
            if armed:
                assert lib.moe_grouped_ffn_time_next_call(events) == 0
            rc, names = step(ints)
            assert rc == 0
            print(sum("grouped_" in n for n in names), sum("grouped_ffn_tiles" in n for n in names))
    """)
    assert out.split("\n")[:3] == ["1 1", "2 0", "1 1"], out


def test_shapes_of_the_shared_launch_reach_it(child):
    """The shapes that tests/test_gpu_ffn.py holds against a launch each are of the form that they are listed as."""
    from test_gpu_ffn import ONE_LAUNCH
    child(f"""
        c_p = ctypes.c_void_p
        X, OF, GATE_W, SEG, SLOT, PACKED, Y, WS = [i << 40 for i in range(1, 9)]
        plain = [c_p, c_int, c_i64] + [c_int] * 3 + [c_p] * 2 + [c_int] * 3 + [c_p] * 3 + [c_sz, c_p]
        fused = [c_p] + [c_int] * 3 + [c_p] * 2 + [c_int] * 3 + [c_p] * 2 + [c_int] * 3 + [c_p] * 3 + [c_sz, c_p]
        for f in (lib.moe_grouped_ffn, lib.moe_grouped_ffn_relu):
            f.argtypes = plain
        lib.moe_grouped_ffn_fused.argtypes = fused
        for d, swiglu, relu, sizes, both in {ONE_LAUNCH}:
            e, a = len(sizes), sum(sizes) // 2 * 2
            for form, ffn in (("plain", swiglu), ("relu", relu), ("gather", swiglu), ("weights", swiglu)):
                tail = (SEG, SLOT, e + 2, 0, e + 2, PACKED, Y, WS, lib.moe_grouped_ffn_workspace_bytes(a, d, ffn, e + 2, 1), None)
                for group_n in (0, 4):
                    assert lib.moe_grouped_ffn_set_option(3, group_n) == 0
                    rt.start(HOOK())
                    if form in ("plain", "relu"):
                        rc = (lib.moe_grouped_ffn if form == "plain" else lib.moe_grouped_ffn_relu)(X, 1, a, d, ffn, e, *tail)
                    else:
                        rc = lib.moe_grouped_ffn_fused(X, 1, a // 2, 2, OF, GATE_W if form == "weights" else None, d, ffn, e, *tail)
                    names = rt.launches().decode()
                    assert rc == 0 and ("grouped_ffn_tiles" in names) == (both and group_n == 0), (d, ffn, sizes, form, rc, names)
    """)
