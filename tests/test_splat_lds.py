"""Every splat tile that the tuning cache accepts has to launch: the kernels' static LDS and the
largest dynamic LDS that the check of a tile allows make up the 160 KB of a CU at most.  The
static LDS is read from the kernel metadata of the library that was built."""

from paper_2601_22793_amd import _lib as L

LDS = 160 * 1024


def uint_at(b, i):
    """The MessagePack unsigned integer at offset i."""
    tag = b[i]
    if tag < 0x80:
        return tag
    n = {0xcc: 1, 0xcd: 2, 0xce: 4}[tag]
    return int.from_bytes(b[i + 1:i + 1 + n], "big")


def str_at(b, i):
    """The MessagePack string at offset i."""
    tag = b[i]
    if tag & 0xe0 == 0xa0:
        n, i = tag & 0x1f, i + 1
    else:
        w = {0xd9: 1, 0xda: 2}[tag]
        n, i = int.from_bytes(b[i + 1:i + 1 + w], "big"), i + 1 + w
    return b[i:i + n].decode()


def static_lds():
    blob = open(L.LIB_PATH, "rb").read()
    key, name = b".group_segment_fixed_size", b"\xa5.name"
    out = {}
    i = blob.find(key)
    while i >= 0:
        j = blob.find(name, i) + len(name)
        out[str_at(blob, j)] = uint_at(blob, i + len(key))
        i = blob.find(key, i + 1)
    return out


def test_accepted_tiles_fit_in_lds():
    splat = {k: v for k, v in static_lds().items() if "k_splat" in k}
    assert len(splat) >= 16
    # the same limit as in epr_autotune's check: the accumulators of at most 160 KB - 64 bytes
    biggest = max(4 * n * (tx + 2) * (ty + 2) for n in range(1, L.EPR_MAX_LINES + 1)
                  for tx in range(8, 257) for ty in range(8, min(256, 4096 // tx) + 1)
                  if 4 * n * (tx + 2) * (ty + 2) <= LDS - 64)
    for k, v in splat.items():
        assert v + biggest <= LDS, (k, v, biggest)
