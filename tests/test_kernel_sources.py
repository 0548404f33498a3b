"""Rules of the kernel sources that no run can show to be broken: code that breaks them may pass every test."""
import math
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1410_7455_amd", "csrc")


def sources():
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            yield name, re.sub(r"//[^\n]*", "", f.read())


def test_wavefront_barriers_are_fenced():
    """A wave barrier does not order memory for the compiler: lanes that exchange data through LDS need a release before it
    and an acquire behind it."""
    fenced = (r'__builtin_amdgcn_fence\(__ATOMIC_RELEASE, "wavefront"\);\s*__builtin_amdgcn_wave_barrier\(\);\s*'
              r'__builtin_amdgcn_fence\(__ATOMIC_ACQUIRE, "wavefront"\);')
    seen = 0
    for name, text in sources():
        all_of_them = len(re.findall(r"__builtin_amdgcn_wave_barrier\(\)", text))
        assert all_of_them == len(re.findall(fenced, text)), name
        seen += all_of_them
    assert seen > 0


def test_no_load_in_inline_assembly():
    """The compiler takes the output of an assembly statement as written at once: with the wait in another statement it
    may use or reuse the register while the load is in flight."""
    for name, text in sources():
        assert not re.search(r'asm[^;]*"[^"]*(global|buffer|flat|ds|s)_(load|read)', text), name


def tile_tables():
    """The constants of the layer products' tile choice, as the library is built with them."""
    with open(os.path.join(CSRC, "ngsgd.hip")) as f:
        text = f.read()

    def table(name):
        body = re.search(name + r"\[[^=]*=\s*(\{.*?\});", text, re.S).group(1)
        return eval(body.replace("{", "[").replace("}", "]"), {"__builtins__": {}})

    def number(name):
        return float(re.search(name + r" = ([0-9.]+);", text).group(1))

    tiles = re.search(r"enum LayerTile \{([^}]*)\}", text).group(1).replace(" ", "").split(",")[:-1]
    return dict(tiles=tiles, bm=table("kTileBM"), bn=table("kTileBN"), fill=table("kTileFill"), resident=table("kTileResident"),
                block=table("kTileBlock"), launch=number("kTileLaunch"), units=int(number("kComputeUnits")),
                slabs=int(number("kMaxBwdSplits")), target=int(number("kTargetBlocks")))


FORWARD, BACKWARD, UPDATE = range(3)


def tile_of(t, layout, products):
    """The choice of pick_layer_tile for products (M, N, K, splits) of one launch."""
    best = None
    for i, name in enumerate(t["tiles"]):
        if name == "TILE_64x64" and layout != FORWARD:
            continue
        tiles, depth = 0, 0.0
        for m, n, k, splits in products:
            here = -(-m // t["bm"][i]) * -(-n // t["bn"][i]) * splits
            tiles += here
            depth += here * -(-k // splits)
        rounds = -(-tiles // t["units"])
        cost = (t["launch"] + math.ceil(rounds / t["resident"][i]) * t["fill"][i] +
                rounds * math.ceil(depth / tiles / 64.0) * t["block"][layout][i])
        if best is None or cost < best[0]:
            best = (cost, name)
    return best[1]


def tiles_of_network(t, n, din, hidden, classes):
    """(layout, tile) of every layer product that test_gradients_of_a_plain_network launches for one of its shapes."""
    layers = [(din + 1, hidden), (hidden + 1, classes)]
    out = {(FORWARD, tile_of(t, FORWARD, [(n, o, i, 1)])) for i, o in layers}
    slabs = t["target"] // (-(-n // 64) * -(-hidden // 64))
    out.add((BACKWARD, tile_of(t, BACKWARD, [(n, hidden, classes, min(t["slabs"], max(1, min(slabs, -(-classes // 32)))))])))
    out.add((UPDATE, tile_of(t, UPDATE, [(o, i, n, 1) for i, o in layers])))
    out |= {(UPDATE, tile_of(t, UPDATE, [(o, i, n, 1)])) for i, o in layers}   # last_gradient: one product a launch
    return out


def test_layer_product_tests_reach_every_tile():
    """The shapes of the layer products' tests select every tile that is built for a layout."""
    from test_gpu_layer_products import SHAPES
    t = tile_tables()
    reached = set().union(*(tiles_of_network(t, *shape) for shape in SHAPES))
    built = {(layout, name) for layout in range(3) for name in t["tiles"] if name != "TILE_64x64" or layout == FORWARD}
    assert built == reached


def test_traffic_summary_lists_the_layer_products():
    """bench.py reports the HBM traffic of a layer product from the committed counter summary: the summary has to be of the
    kernels that are launched."""
    import bench
    for category in ("gemm_fwd", "gemm_bwd", "gemm_upd"):
        traffic = bench.measured_traffic_per_launch(category)
        assert traffic is not None and 1e6 < traffic < 1e9, category
    assert bench.measured_traffic_per_launch("elementwise") is None


def enclosing(text, at):
    """What stands in front of the braces around a position, innermost first: the conditions under which it runs."""
    depth, out = 0, []
    for i in range(at, -1, -1):
        if text[i] == "}":
            depth += 1
        elif text[i] == "{":
            if depth == 0:
                out.append(re.split(r"[;{}]", text[:i])[-1].strip())
            depth = max(depth - 1, 0)
    return out


def test_workgroups_of_an_eigen_update_decide_alike():
    """Every workgroup of an instance decides for itself whether the direct solver served, and writes its rows of A_t or leaves
    them to the first one: what they compare with the limits has to be the same numbers in all of them, so no comparison may
    depend on which workgroup makes it."""
    text = dict(sources())["small_update.h"]
    body = text[text.index("void eig_finish_kernel"):text.index("__syncthreads_or(bad")]
    comparisons = [m.start() for m in re.finditer(r"bad \|=", body)]
    assert len(comparisons) >= 4
    for at in comparisons:
        conditions = enclosing(body, at) + [re.split(r"[;{}]", body[:at])[-1]]
        assert not any(re.search(r"blockIdx|first_row|lead", c) for c in conditions), conditions


def test_deferred_count_is_read_before_the_ticket():
    """The last workgroup of an instance clears the number of deferred patches, by which every wavefront of every workgroup chooses
    its way: a workgroup takes its ticket only behind a barrier that all of its wavefronts reach with the number in hand."""
    text = dict(sources())["kernels.h"]
    kernel = text[text.index("void finish_apply_kernel"):]
    assert "a.deferred_count()" in kernel[:kernel.index("finish_deferred<SCALE>")] and "a.ticket()" not in kernel
    way = text[text.index("void finish_deferred"):text.index("void finish_apply_kernel")]
    assert way.index("__syncthreads();") < way.index("a.ticket()") < way.index("a.left()") < way.index("a.arrive + i, 0")


def test_every_tile_of_the_elimination_has_one_workgroup():
    """simple_sweep_kernel deals the tiles on and above the diagonal to a grid that is made for the largest matrix of its group: with
    the kernel's own rules every tile of a smaller one is met once too."""
    text = dict(sources())["simple_ng.h"]
    body = text[text.index("void simple_sweep_kernel"):]
    body = body[:body.index("__shared__")]
    rules = ["int ty = blockIdx.y, tx = ty + (int)blockIdx.x - 1;", "const int over = tx - tiles;", "ty = tiles - 1 - ty;", "tx = ty + over;",
             "if (ty <= (int)blockIdx.y) return;", "if (!ahead && tx >= tiles) return;"]
    assert all(r in body for r in rules)
    dropped = re.search(r"if \(k >= nblk \|\| (.*)\) return;", body).group(1).replace("(int)blockIdx.y", "y")
    for largest in range(1, 18):
        for tiles in range(1, largest + 1):
            met = []
            for y in range((largest + 1) // 2):
                for x in range(1, largest + 2):
                    ty, tx = y, y + x - 1
                    if tx >= tiles:
                        over, ty = tx - tiles, tiles - 1 - ty
                        tx = ty + over
                        if ty <= y:
                            continue
                    if eval(dropped, {"__builtins__": {}}, dict(y=y, tiles=tiles)) or tx >= tiles:
                        continue
                    met.append((ty, tx))
            assert sorted(met) == [(i, j) for i in range(tiles) for j in range(i, tiles)], (largest, tiles)


def test_wide_patches_leave_no_dies_idle():
    """The fused apply kernel's patches of 320 columns: four narrow ones per compute unit, and a busiest die with at most three
    quarters of the work.  The shapes of their test that are meant to take them do."""
    from test_gpu_fused_apply import WIDE
    text = dict(sources())["ngsgd.hip"]
    number = {n: int(re.search(n + r" = (\d+);", " ".join(t for _, t in sources())).group(1))
              for n in ("kFusedWideUnits", "kFusedChunk", "kFusedWide", "kFusedRows", "kXcds")}
    assert "return 4 * busiest_die(list, done, n, kFusedWide) <= 3 * busiest_die(list, done, n, kFusedChunk) ? kFusedWide : kFusedChunk;" in text

    def busiest(n, d, columns):   # of one matrix
        load = [0] * number["kXcds"]
        for c in range(-(-d // columns)):
            load[c % number["kXcds"]] += -(-n // number["kFusedRows"])
        return max(load)

    wide = {(n, d, r): r > 32 and -(-n // number["kFusedRows"]) * -(-d // number["kFusedChunk"]) > number["kFusedWideUnits"] and
            4 * busiest(n, d, number["kFusedWide"]) <= 3 * busiest(n, d, number["kFusedChunk"]) for n, d, r in WIDE + [(2048, 5000, 80), (512, 5000, 80)]}
    assert [k for k in wide if wide[k]] == [(4033, 2497, 41), (1990, 5001, 96), (4096, 2401, 80), (4090, 2560, 33), (2048, 5000, 80)]
