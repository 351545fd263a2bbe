"""Plan files whose checksums are right but whose tables do not fit the plan
they describe (a faulty writer): refused with SHT_ECORRUPT, since loading
indexes host memory and the kernels index device memory with those values.
Files are taken apart, changed and signed again here; host-only, no GPU.
"""
import struct

import numpy as np
import pytest

MASK = (1 << 64) - 1
HEADER = 152  # bytes; the last eight are the header's own hash, payload hash at 24
P1, P2 = 0x9E3779B97F4A7C15, 0xC2B2AE3D27D4EB4F
BLOCK = 16 << 20

# the fields of a brute-force plan in file order: scalars by their struct
# code, tables by their numpy type
BRUTE = ["nrings i", "n_north i", "n_north_pad i", "n_dd_pad i", "n_dd_rings i", "n_dd_groups i", "rings_per_lane i",
         "ring_threads i", "n_step q", "n_step_exec q", "n_step_dd q", "n_step_lanes q", "tw_log i", "build_seconds d",
         "z2_hi f8", "z2_lo f8", "ring_J i4", "ring_s i4", "ring_off i8", "coef_off i8", "coef_hi f8", "coef_lo f8",
         "start_idx i4", "start_val f8", "start_lo f8", "grp_lo i4", "grp_hi i4", "tw f8", "ring_M i4",
         "ring_bs_off i8", "bs_table f8", "chirp f8", "ring_chirp_off i8", "pol_n i", "pol_ring f8", "pol_K f8",
         "classes Q"]
CLASS = ["lds_entries i", "wrap i", "rings i4"]
BFLY = ["K i", "ws_entries q", "max_n i", "depth i4", "n_tasks q", "res_task i4", "res_lane i4", "res_val f8",
        "res_sub i4", "nbatch i", "batch_count i4", "batch_task i8", "batch_sub i8", "lv_off i8", "lv_max_n i4",
        "perm i2", "node_i i4", "T f8", "T_entries q", "res_elems q", "n_nodes q", "n_res_lanes q", "n_units q",
        "level_T 11q", "level_units 11q", "level_nodes 11q", "f1_unit i4", "l1_plain i4", "fold_slot i4", "f1_off i8",
        "l1_off i8", "fold_off i8", "res_exec q", "depth_hist 11q", "bf_build_seconds d"]


def mix64(x):
    x ^= x >> 30
    x = x * 0xBF58476D1CE4E5B9 & MASK
    x ^= x >> 27
    x = x * 0x94D049BB133111EB & MASK
    return x ^ x >> 31


def rotl(x, r):
    return (x << r | x >> (64 - r)) & MASK


def hash_bytes(b, seed):
    n = len(b)
    h = [seed ^ P1, seed ^ P2, (seed + P1) & MASK, (seed - P2) & MASK]
    words = struct.unpack(f"<{n // 8}Q", b[:n // 8 * 8])
    whole = n // 32 * 4
    for i in range(0, whole, 4):
        for j in range(4):
            h[j] = rotl(h[j] ^ (words[i + j] * P1 & MASK), 31) * P2 & MASK
    rest = list(words[whole:])
    if n % 8:
        rest.append(int.from_bytes(b[n // 8 * 8:], "little"))
    for w in rest:
        h[0] = rotl(h[0] ^ (w * P1 & MASK), 31) * P2 & MASK
    return mix64(h[0]) ^ rotl(mix64(h[1]), 16) ^ rotl(mix64(h[2]), 32) ^ rotl(mix64(h[3]), 48) ^ n


class File:
    """A plan file as named pieces; save() signs it again."""

    def __init__(self, path):
        data = open(path, "rb").read()
        self.header, self.pieces, self.at = bytearray(data[:HEADER]), [], {}
        pos = HEADER

        def take(name, nbytes):
            nonlocal pos
            self.at[name] = len(self.pieces)
            self.pieces.append(data[pos:pos + nbytes])
            pos += nbytes
            return self.pieces[-1]

        def fields(names, tag=""):
            for f in names:
                name, kind = f.split()
                if kind[0] == "f" or (kind[0] == "i" and len(kind) > 1):
                    n, = struct.unpack("<Q", take(tag + name + ".size", 8))
                    take(tag + name, n * int(kind[1]))
                else:
                    take(tag + name, struct.calcsize("<" + kind))
        fields(BRUTE)
        for c in range(struct.unpack("<Q", self.pieces[self.at["classes"]])[0]):
            fields(CLASS, f"class{c}.")
        assert struct.unpack("<i", take("interp", 4)) == (0,)
        if struct.unpack("<i", take("butterfly", 4))[0]:
            fields(BFLY)
        assert pos == len(data)

    def array(self, name, dtype):
        return np.frombuffer(self.pieces[self.at[name]], dtype).copy()

    def put(self, name, value):
        self.pieces[self.at[name]] = value.tobytes() if isinstance(value, np.ndarray) else value
        if name + ".size" in self.at:
            self.pieces[self.at[name + ".size"]] = struct.pack("<Q", len(value))

    def save(self, path):
        units = []
        for p in self.pieces:
            units += [p[o:o + BLOCK] for o in range(0, len(p), BLOCK)] or [p]
        h = 0x243F6A8885A308D3
        for i, u in enumerate(units):
            h = mix64(((h ^ hash_bytes(u, i)) + P1) & MASK)
        head = bytearray(self.header)
        struct.pack_into("<QQ", head, 16, sum(map(len, self.pieces)), h)
        struct.pack_into("<Q", head, HEADER - 8, hash_bytes(bytes(head[:HEADER - 8]), 0x5A5A5A5A))
        with open(path, "wb") as f:
            f.write(head)
            for p in self.pieces:
                f.write(p)


@pytest.fixture(scope="module")
def sht():
    from paper_1110_4874_amd import sht as mod
    mod.load()
    return mod


@pytest.fixture(scope="module")
def brute(sht, tmp_path_factory):
    path = str(tmp_path_factory.mktemp("plans") / "b.plan")
    sht.Plan(40, 12, host_only=True).save(path)  # rings of 24 pixels' half length 12 and powers of two
    return path


def test_signing_reproduces_the_file(sht, brute, tmp_path):
    again = str(tmp_path / "again.plan")
    File(brute).save(again)
    assert open(brute, "rb").read() == open(again, "rb").read()


def refused(sht, f, tmp_path):
    bad = str(tmp_path / "bad.plan")
    f.save(bad)
    with pytest.raises(sht.ShtError) as e:
        sht.Plan.load(bad, host_only=True)
    assert e.value.code == sht.SHT_ECORRUPT and "inconsistent" in str(e.value), str(e.value)


def changed(name, dtype, index, value):
    def change(f):
        a = f.array(name, dtype)
        a[index] = value
        f.put(name, a)
    return change


def cut(name, dtype):
    return lambda f: f.put(name, f.array(name, dtype)[:-1])


# nside 12: ring 0 has half length 2, ring 4 half length 10 (Bluestein, 16 points)
@pytest.mark.parametrize("change", [
    changed("ring_M", "i4", 4, 8192), changed("ring_M", "i4", 4, 8), changed("ring_M", "i4", 4, 24),
    changed("ring_M", "i4", 4, -16), changed("ring_M", "i4", 4, 0), changed("ring_M", "i4", 0, 16),
    changed("ring_bs_off", "i8", 4, 1 << 40), changed("ring_bs_off", "i8", 4, -1), cut("ring_bs_off", "i8"),
    changed("ring_chirp_off", "i8", 4, 1 << 40), changed("ring_chirp_off", "i8", 4, -1), cut("ring_chirp_off", "i8"),
    cut("bs_table", "f8"), cut("chirp", "f8"), changed("ring_J", "i4", 4, 1 << 20), changed("ring_off", "i8", 4, 1 << 40),
    changed("ring_s", "i4", 4, 7), changed("tw_log", "i4", 0, 13), changed("tw_log", "i4", 0, 0),
], ids=range(19))
def test_ring_tables(sht, brute, tmp_path, change):
    f = File(brute)
    change(f)
    refused(sht, f, tmp_path)


# L = 40, nside 12: 24 north rings in 64 lanes; order 0 has 41 + 24 coefficients (66 with padding)
@pytest.mark.parametrize("change", [
    changed("coef_off", "i8", 0, 2), changed("coef_off", "i8", 5, 1 << 40), changed("coef_off", "i8", 5, -4),
    changed("start_idx", "i4", 0, -8), changed("start_idx", "i4", 0, 4), changed("start_idx", "i4", 0, 24),
    changed("start_idx", "i4", 63, 0x3FFFFFFE), changed("start_idx", "i4", -1, 0),
    changed("grp_lo", "i4", 0, -8), changed("grp_lo", "i4", 3, 8), changed("grp_hi", "i4", 0, 1 << 20), cut("grp_hi", "i4"),
    changed("n_dd_groups", "i4", 0, 1), changed("n_dd_groups", "i4", 0, -1), changed("n_dd_pad", "i4", 0, 64),
    changed("n_dd_rings", "i4", 0, 25), cut("start_lo", "f8"), cut("z2_lo", "f8"),
], ids=range(18))
def test_chain_tables(sht, brute, tmp_path, change):
    f = File(brute)
    change(f)
    refused(sht, f, tmp_path)


@pytest.fixture(scope="module")
def compressed(sht, tmp_path_factory):
    path = str(tmp_path_factory.mktemp("plans") / "c.plan")
    p = sht.Plan(47, 12, 1e-6, max_levels=1, host_only=True)
    assert p.info()["bf_depth_hist"][1] > 0
    p.save(path)
    return path


@pytest.mark.parametrize("change", [
    changed("f1_off", "i8", 0, -1), changed("f1_off", "i8", -1, 1 << 40), cut("f1_off", "i8"), cut("f1_unit", "i4"),
    changed("l1_off", "i8", -1, 1 << 40), changed("fold_off", "i8", 0, 1),
    changed("res_lane", "i4", 1, -8), changed("res_lane", "i4", 0, 24), changed("res_lane", "i4", 0, -1),
], ids=range(9))
def test_compressed_tables(sht, compressed, tmp_path, change):
    f = File(compressed)
    change(f)
    refused(sht, f, tmp_path)
