"""One scenario a process: libmlpmoe.so on the recorded runtime of fake_hip.cpp.  argv: scenario, fake library, library."""
import ctypes
import sys

fake = ctypes.CDLL(sys.argv[2], ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[3])
fake.fake_record.restype = ctypes.c_char_p
fake.fake_largest_allocation.argtypes = [ctypes.c_size_t]
lib.mlpmoe_workspace_bytes.restype = ctypes.c_size_t
lib.mlpmoe_last_error_detail.restype = ctypes.c_char_p
OK, ERR_WORKSPACE, ERR_HIP = 0, -5, -6
P = ctypes.c_void_p(0x10000)                       # any aligned device address: no kernel runs


def record():
    """What the runtime was asked since the last look: [verb, words ...] per call."""
    lines = [l.split() for l in fake.fake_record().decode().splitlines()]
    fake.fake_clear()
    return lines


def verbs(lines):
    return [l[0] for l in lines]


def kernels(lines):
    return [l[1] for l in lines if l[0] == "launch"]


def table(widths, mask=None):
    n = len(widths)
    off = (ctypes.c_int32 * (n + 1))()
    for b, w in enumerate(widths):
        off[b + 1] = off[b] + w
    return off, (ctypes.c_float * n)(*[1.0] * n), (ctypes.c_uint8 * n)(*(mask or [1] * n)), off[n], n


def forward(f, T, d_model, widths, mask=None, route=False):
    off, alpha, on, d_inter, B = table(widths, mask)
    args = [P, P, P, P, off, alpha, on] + ([P] if route else []) + [T, d_model, d_inter, B, P, None]
    return f(*args)


def least_and_full(T, d_model, d_inter, B):
    """Float storage: the workspace without the partial sums of a K split (H, the tile tables, the slack: what the bf16
    call of a size that never splits has, with H twice as large) and with them."""
    full = lib.mlpmoe_workspace_bytes(T, d_model, d_inter, B, 4)
    ld = lib.mlpmoe_hidden_ld(d_inter)
    hidden2, hidden4 = ((T * ld * e + 255) // 256 * 256 for e in (2, 4))
    wide = lib.mlpmoe_workspace_bytes(T, 1 << 22, d_inter, B, 2)     # so many output tiles that K is never split
    return wide - hidden2 + hidden4, full


def graph_block_stays():
    """A block that a recorded graph may point into is replaced only by a call that cannot run in it."""
    T, d_model, widths = 64, 256, [1024] * 4
    least, full = least_and_full(T, d_model, 4096, 4)
    assert least < full, (least, full)
    # a bf16 call leaves a block between the two
    rows = next(t for t in range(T, 4096) if least <= lib.mlpmoe_workspace_bytes(t, d_model, 4096, 4, 2) < full)
    assert forward(lib.mlpmoe_forward_bf16, rows, d_model, widths) == OK
    assert verbs(record()).count("malloc") == 1
    fake.fake_capturing(1)
    assert forward(lib.mlpmoe_forward_f32, T, d_model, widths) == OK           # recorded: runs in what is there
    captured = record()
    fake.fake_capturing(0)
    assert forward(lib.mlpmoe_forward_f32, T, d_model, widths) == OK           # the same call, eager
    eager = record()
    assert "free" not in verbs(captured) + verbs(eager), eager
    assert kernels(captured) == kernels(eager), (captured, eager)
    # a larger call does replace it, and a fresh block has room for the partial sums
    fake.fake_capturing(1)
    assert forward(lib.mlpmoe_forward_f32, 40 * T, d_model, widths) == ERR_WORKSPACE
    assert not record()
    fake.fake_capturing(0)
    lib.mlpmoe_release()
    record()
    assert forward(lib.mlpmoe_forward_f32, T, d_model, widths) == OK
    assert record()[0] == ["malloc", str(full)]


def short_of_memory():
    """A float call or plan takes the block without room for partial sums where there is no memory for the larger one."""
    T, d_model, widths = 64, 256, [1024] * 4
    least, full = least_and_full(T, d_model, 4096, 4)
    off, alpha, on, d_inter, B = table(widths)
    plan = ctypes.c_void_p()
    fake.fake_largest_allocation(full - 1)
    assert forward(lib.mlpmoe_forward_f32, T, d_model, widths) == OK
    assert lib.mlpmoe_plan_create(off, alpha, on, d_model, d_inter, B, 4, T, ctypes.byref(plan)) == OK
    assert lib.mlpmoe_plan_forward(plan, P, P, P, P, T, P, None) == OK
    assert [l for l in record() if l[0] == "malloc"] == [["malloc", str(least)]] * 2
    assert lib.mlpmoe_plan_destroy(plan) == OK and lib.mlpmoe_release() == OK
    # no memory for that either: refused, and nothing launched
    record()
    fake.fake_largest_allocation(least - 1)
    assert forward(lib.mlpmoe_forward_f32, T, d_model, widths) == ERR_WORKSPACE
    assert lib.mlpmoe_plan_create(off, alpha, on, d_model, d_inter, B, 4, T, ctypes.byref(plan)) == ERR_HIP and not plan
    assert verbs(record()) == ["refuse"] * 4


def most_tokens():
    """Tables with odd boundaries and float storage end where the generic kernels' grid ends."""
    most = 65535 * 64
    widths, on = [131, 133], [1, 0]
    for f, route in ((lib.mlpmoe_forward_bf16, False), (lib.mlpmoe_forward_bf16_out_bf16, False),
                     (lib.mlpmoe_forward_routed_bf16, True), (lib.mlpmoe_forward_f32, False)):
        assert forward(f, most, 8, widths, on, route) == OK
        assert any("gate_up_mfma" in k for k in kernels(record()))
        assert forward(f, most + 1, 8, widths, on, route) == ERR_HIP
        assert "invalid argument" in lib.mlpmoe_last_error_detail().decode()
        assert not kernels(record())


def widest_routed():
    """Odd boundaries, routed, on the widest layers: the generic kernels take what the tile list does not hold."""
    on = [1, 0] * 31 + [1, 1]
    for width, kernel in ((1 << 22, "gate_up_generic"), ((1 << 22) - 64 * 128, "gate_up_mfma_routed")):
        for T in (1, 300):
            widths = [9, 23] * 31 + [width - 31 * 32 - 1, 1]            # a tile of its own for each short run
            assert forward(lib.mlpmoe_forward_routed_bf16, T, 8, widths, on, True) == OK, lib.mlpmoe_last_error_detail()
            assert any(kernel in k for k in kernels(record())), (width, T)


def smallest_routed():
    """Odd boundaries, routed, on the smallest layers: two launches of the generic kernels, not three or four."""
    for d_model, width, kernel in ((8, 64, "gate_up_generic"), (8, 240, "gate_up_generic"), (8, 248, "gate_up_mfma_routed"),
                                   (128, 128, "gate_up_mfma_routed")):
        for T in (1, 1000):
            assert forward(lib.mlpmoe_forward_routed_bf16, T, d_model, [13, width - 13], None, True) == OK
            assert any(kernel in k for k in kernels(record())), (d_model, width, T)


def unsplit_narrow():
    """Narrow layers with many tokens, 17 to 32 K tiles: the down projection fills the chip unsplit and stays so."""
    for d_model, d_inter, T, split in ((448, 1408, 3565, False), (320, 1088, 3088, False), (512, 2048, 4096, False),
                                       (640, 1600, 1684, True)):        # too few tiles: split
        assert forward(lib.mlpmoe_forward_bf16, T, d_model, [d_inter]) == OK
        assert any("reduce_partials" in k for k in kernels(record())) == split, (d_model, d_inter, T)


def in_place():
    """A result over x: the decode gate+up kernel, whose workgroups read all of x, does not clear it; a launch behind it does."""
    ptr = ctypes.c_void_p
    for f, x, out, n in ((lib.mlpmoe_forward_f32, 1 << 20, 1 << 20, 3), (lib.mlpmoe_forward_f32, 1 << 20, (1 << 20) + 16, 3),
                         (lib.mlpmoe_forward_f32, 1 << 20, (1 << 20) - 16, 3), (lib.mlpmoe_forward_bf16, 1 << 20, 1 << 20, 3),
                         (lib.mlpmoe_forward_f32, 1 << 20, (1 << 20) + 8 * 256 * 4, 2),
                         (lib.mlpmoe_forward_f32, 1 << 20, (1 << 20) - 8 * 256 * 4, 2),
                         (lib.mlpmoe_forward_f32, 1 << 20, 2 << 20, 3), (lib.mlpmoe_forward_f32, 1 << 20, 3 << 20, 3)):
        for widths in ([128, 128], [101, 155]):
            off, alpha, on, d_inter, B = table(widths, [1, 0])
            # W_gate and W_up at 2 and 3 MiB
            assert f(ptr(x), ptr(2 << 20), ptr(3 << 20), ptr(8 << 20), off, alpha, on, 8, 256, d_inter, B, ptr(out), None) == OK
            names = kernels(record())
            assert len(names) == n and "gate_up_once" in names[0] and "down_rows" in names[-1], names
            assert n == 2 or "fill_zero" in names[1], names


def decode_gate_up():
    """The one-tile gate+up kernel where all its workgroups together load little of x, the ring kernel elsewhere."""
    for T, d_model, d_inter, once in ((1, 896, 4864, 1), (8, 896, 4864, 1), (16, 896, 4864, 1), (16, 1024, 5504, 1), (8, 1536, 8192, 1),
                                      (9, 1024, 4096, 1), (9, 1032, 4096, 0), (10, 1152, 6208, 0), (12, 1280, 6912, 0),
                                      (8, 1536, 10880, 1), (8, 1536, 11008, 0), (8, 1280, 32768, 0), (16, 896, 8192, 0),
                                      (4, 896, 65536, 1), (1, 1544, 1024, 0)):
        assert forward(lib.mlpmoe_forward_bf16, T, d_model, [d_inter]) == OK, lib.mlpmoe_last_error_detail()
        name = kernels(record())[0]
        assert ("gate_up_once" if once else "gate_up_xreg") in name, (T, d_model, d_inter, name)
    for T, d_model, once in ((12, 1152, 1), (8, 1536, 1), (16, 896, 1), (16, 904, 0), (1, 1544, 0)):     # routed: by x alone
        assert forward(lib.mlpmoe_forward_routed_bf16, T, d_model, [16384], None, True) == OK
        assert ("gate_up_once" if once else "gate_up_xreg") in kernels(record())[0], (T, d_model)


def decode_few_tokens():
    """One or two tokens: fewer rows per workgroup, with a bf16 result and on every wide layer."""
    f32, b16 = lib.mlpmoe_forward_bf16, lib.mlpmoe_forward_bf16_out_bf16
    rows8, rows4 = "down_rowsILi8ELi5ELi8", "down_rowsILi8ELi5ELi4"
    for f, T, d_model, kernel in ((f32, 1, 4096, rows8), (f32, 2, 4096, rows8), (f32, 3, 4096, "down_split"), (f32, 1, 16384, rows8),
                                  (b16, 1, 1152, rows4), (b16, 2, 2056, rows4), (b16, 3, 1152, rows8),
                                  (b16, 2, 8192, rows4), (b16, 3, 4096, "decode_kernel")):
        assert forward(f, T, d_model, [1024]) == OK, lib.mlpmoe_last_error_detail()
        name = kernels(record())[-1]
        assert kernel in name, (T, d_model, name)
    for T, d_model, kernel in ((2, 4096, "down_splitILi4"), (1, 8192, "down_splitILi4"), (1, 4096, rows8), (2, 3056, rows8)):
        assert forward(lib.mlpmoe_forward_routed_bf16, T, d_model, [1024], None, True) == OK
        assert kernel in kernels(record())[-1], (T, d_model)


def decode_down():
    """Narrow layers with a long K: the 16-wave kernel adds up the halves; all others as before it."""
    for T, d_model, d_inter, kernel in ((8, 1280, 12288, "down_rows"), (8, 1280, 12352, "down_splitILi16"), (16, 1280, 8128, "down_rows"),
                                        (16, 1280, 8192, "down_splitILi16"), (1, 1032, 16384, "down_splitILi16"), (16, 1024, 32768, "down_rows"),
                                        (8, 2056, 32768, "down_rows"), (16, 2560, 12288, "down_rows"), (16, 2560, 12296, "down_splitILi16"),
                                        (16, 3064, 16384, "down_splitILi4")):
        assert forward(lib.mlpmoe_forward_bf16, T, d_model, [d_inter]) == OK, lib.mlpmoe_last_error_detail()
        name = kernels(record())[-1]
        assert kernel in name, (T, d_model, d_inter, name)
        assert forward(lib.mlpmoe_forward_bf16_out_bf16, T, d_model, [d_inter]) == OK
        assert "down_split" not in kernels(record())[-1]
    assert forward(lib.mlpmoe_forward_routed_bf16, 8, 1280, [16384], None, True) == OK       # how long K is depends on the routes
    assert "down_rows" in kernels(record())[-1]


def decode_odd_boundaries():
    """Tables with odd boundaries and so many active neurons that the prefill kernels fill the chip stay on those."""
    for T, d_model, active, rows in ((16, 896, 8191, 1), (9, 896, 8193, 0), (16, 1600, 8191, 1), (8, 1280, 32767, 1), (8, 1280, 32769, 0),
                                     (4, 1280, 49157, 1), (1, 2048, 49157, 1), (13, 2048, 1001, 0), (17, 512, 1001, 0)):
        for f in (lib.mlpmoe_forward_bf16, lib.mlpmoe_forward_bf16_out_bf16):
            assert forward(f, T, d_model, [active, 8 - active % 8 + 64], [1, 0]) == OK, lib.mlpmoe_last_error_detail()
            name = kernels(record())[0]
            assert ("gate_up_once" if rows else "gate_up_mfma") in name, (T, d_model, active, name)


def routed_grid():
    """The routed gate+up kernel has few more workgroups than there are tiles, and a grid that can be launched at the most tokens."""
    for T, d_model, widths in ((3000, 3072, [1120] * 16), (1 << 24, 8, [136, 8] * 32)):
        on = [1, 0] * 32 if len(widths) == 64 else None
        assert forward(lib.mlpmoe_forward_routed_bf16, T, d_model, widths, on, True) == OK, lib.mlpmoe_last_error_detail()
        name, grid = next((l[1], int(l[2])) for l in record() if l[0] == "launch" and "gate_up_mfma_routed" in l[1])
        tiles = -(-T // 256) * (64 if on else 140)
        assert tiles + 192 <= grid <= tiles + 300 and grid * 512 < 1 << 32, (T, tiles, grid)


def float_blocks():
    """Float storage in blocks too small for the partial sums of all splits: several splits per workgroup, and where there is room for
    four partial sums (all that was ever asked for at this size before K was split further) still a workgroup for each."""
    T, d_model, widths = 256, 896, [1216] * 4
    least, full = least_and_full(T, d_model, 4864, 4)
    part = T * d_model * 4
    lib.mlpmoe_forward_f32_ws.argtypes = None
    off, alpha, on, d_inter, B = table(widths)
    seen = []
    for n in (full, full - 256, least + 4 * part, least + 2 * part, least):
        assert lib.mlpmoe_forward_f32_ws(P, P, P, P, off, alpha, on, T, d_model, d_inter, B, P, P, ctypes.c_size_t(n), None) == OK
        launches = [l for l in record() if l[0] == "launch"][1:]
        assert "down_mfma" in launches[0][1] and (len(launches) == 1 or "reduce_partials" in launches[1][1]), launches
        seen.append((int(launches[0][2]) // 56, len(launches)))           # 4 x 14 tiles of 64 x 64
    splits = (full - least) // part
    assert splits > 4 and seen == [(splits, 2)] + [(s, 2) for s in (seen[1][0],) * 2] + [(1, 1)] * 2 and 2 < seen[1][0] <= 4, (splits, seen)


def float_token_tiles():
    """Float storage, gate+up: 32-token tiles where they take fewer rounds, and with a deep ring where one round of the chip is enough
    for either and K is long."""
    tile64, tile32, deep = "gate_up_mfmaILi64ELi2ELi1ELi2E", "gate_up_mfmaILi32ELi2ELi1ELi2E", "gate_up_mfmaILi32ELi2ELi1ELi4E"
    for T, d_model, d_inter, kernel in ((20, 896, 4864, deep), (64, 896, 4864, deep), (100, 512, 2560, tile64), (100, 768, 2560, deep),
                                        (100, 764, 2560, tile64), (128, 896, 4864, tile32), (256, 896, 4864, tile64),
                                        (400, 896, 4864, tile32), (330, 512, 2560, tile64)):
        assert forward(lib.mlpmoe_forward_f32, T, d_model, [d_inter]) == OK
        assert kernel in kernels(record())[0], (T, d_model, d_inter)


def partial_sums_at_the_limit():
    """The splits of the calls that test_gpu_split_sum.py has around 16 MiB of partial sums."""
    for T, d_model, d_inter, tile_rows, splits in ((2048, 512, 2048, 128, 4), (1021, 1016, 2048, 128, 4), (1028, 1048, 4096, 256, 5)):
        assert forward(lib.mlpmoe_forward_bf16, T, d_model, [d_inter]) == OK
        _, down, total = [l for l in record() if l[0] == "launch"]
        tiles = -(-T // tile_rows) * -(-d_model // 128)
        assert "down_mfmaILi%dE" % tile_rows in down[1] and "reduce_partials" in total[1], down
        assert int(down[2]) == (tiles * splits + 7) // 8 * 8, (T, down)


globals()[sys.argv[1]]()
print("ok")
