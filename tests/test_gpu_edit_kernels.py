"""The encoder's and decoder's kernels at the sizes where their splits can go
wrong, byte for byte against the oracle: spans of 16384 vertices and waves of
4096 with remainders, fields that start off an alignment boundary, runs of
unchanged spans, the workspace without room for the change bits, varints of
one to ten bytes across payload tiles of 8 KiB, chunks of 4096 entries with a
remainder; and payloads that must be refused."""
import struct

import numpy as np
import pytest
import torch

import paper_2601_01787_amd as pmsz
from oracle import edits
from test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu


def _case(dtype, n, frac, seed, wide=False):
    """fhat and g with a share `frac` of the vertices changed; wide: by up to
    the whole value range (long step counts, raised values too)."""
    rng = np.random.default_rng(seed)
    fhat = (rng.standard_normal(n) * 3).astype(dtype)
    g = fhat.copy()
    m = rng.uniform(size=n) < frac
    if wide:
        g[m] = (rng.standard_normal(m.sum()) * 10.0 ** rng.integers(-20, 20, m.sum())).astype(dtype)
    else:
        g[m] = np.nextafter(g[m], dtype(-np.inf))
    return fhat, g


def _round_trip(fhat, g, off=0, max_edits=None):
    ref = edits.encode(fhat, g)
    n = fhat.size
    a = torch.zeros(n + off, dtype=torch.from_numpy(fhat).dtype, device="cuda")
    b = a.clone()
    a[off:], b[off:] = dev(fhat), dev(g)
    a, b = a[off:].view(1, -1), b[off:].view(1, -1)
    s, ne = pmsz.encode_edits(a, b, max_edits=max_edits)
    assert ne == edits.parse_header(ref)["edits"]
    assert host(s).tobytes() == ref
    back = pmsz.decode_edits(a, s)
    assert np.array_equal(host(back).reshape(-1).view(np.uint8), g.view(np.uint8))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 4095, 4097, 16383, 16384, 16385, 3 * 16384 + 4097])
def test_span_edges(dtype, n):
    for frac in (0.0, 0.02, 1.0):
        fhat, g = _case(dtype, n, frac, n)
        _round_trip(fhat, g, off=n % 3)
    fhat, g = _case(dtype, n, 0.0, n)
    g[0], g[-1] = fhat[0] - 1, fhat[-1] - 1  # the first and the last vertex alone
    _round_trip(fhat, g)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("spans", [3, 513])
def test_spans_with_many_changes(dtype, spans):
    """Words of 64 vertices with up to 64 changes beside empty ones, in grids on
    both sides of 512 spans: listed by lane or by word, written by 512 or 256
    threads."""
    n = spans * 16384 - 77
    rng = np.random.default_rng(spans)
    share = rng.choice([0.0, 0.02, 0.15, 0.3, 0.6, 1.0], size=n // 64 + 1)
    if spans > 3:  # (the oracle takes a second per million entries)
        share[rng.uniform(size=share.size) < 0.9] = 0.0
    fhat = (rng.standard_normal(n) * 3).astype(dtype)
    m = rng.uniform(size=n) < np.repeat(share, 64)[:n]
    g = np.where(m, fhat - dtype(1e-3) * rng.uniform(size=n).astype(dtype), fhat).astype(dtype)
    _round_trip(fhat, g)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_long_gaps_and_no_room_for_the_change_bits(dtype):
    n = 40 * 16384 + 5
    fhat, g = _case(dtype, n, 0.0, 3)
    for i in (16384 * 3 - 1, 16384 * 3, 16384 * 20 + 777, n - 1):
        g[i] = np.nextafter(fhat[i], dtype(-np.inf))
    _round_trip(fhat, g, max_edits=4)
    _round_trip(fhat, g)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("entries", [4095, 4096, 4097, 9000])
def test_wide_steps_across_tiles_and_chunks(dtype, entries):
    fhat, g = _case(dtype, entries, 1.0, entries, wide=True)
    keep = fhat.view(np.uint8).reshape(entries, -1) == g.view(np.uint8).reshape(entries, -1)
    assert not keep.all(axis=1).any()  # every vertex is an entry
    # steps are counted downwards: the oracle's encoder takes lowered values
    lo, hi = np.minimum(fhat, g), np.maximum(fhat, g)
    _round_trip(hi, lo)


def _stream(n, entries, payload, table=None, dt=0):
    """A stream of `entries` entries over n vertices with this payload."""
    nch = (entries + 4095) // 4096
    table = table or [(0, (1 << 64) - 1)] * nch
    return (b"PMSE" + struct.pack("<BBHQQQII", 1, dt, 0, n, entries, len(payload), 4096, nch) +
            b"".join(struct.pack("<QQ", *t) for t in table) + payload)


@pytest.mark.parametrize("what,payload,table", [
    ("no end", b"\x00\x01\x00\x81", None),
    ("one value short", b"\x00\x01\x00", None),
    ("empty", b"", None),
    ("eleven bytes", b"\x00\x01" + b"\x80" * 10 + b"\x00\x01", None),
    ("no step", b"\x00\x01\x00\x00", None),
    ("past the field", b"\x00\x01\x63\x01", None),
    ("gap past the field", b"\x00\x01\x64\x01", None),
    ("huge gap", b"\x00\x01" + b"\xff" * 9 + b"\x01\x01", None),
    ("offset past the payload", b"\x00\x01\x00\x01", [(4, (1 << 64) - 1)]),
    ("offset beyond 63 bits", b"\x00\x01\x00\x01", [(1 << 63, (1 << 64) - 1)]),
    ("previous vertex past the field", b"\x00\x01\x00\x01", [(0, 98)]),
    ("previous vertex beyond 63 bits", b"\x00\x01\x00\x01", [(0, 1 << 63)]),
], ids=lambda v: v.replace(" ", "_") if isinstance(v, str) else "")
def test_malformed_payloads_are_refused(what, payload, table):
    fhat = dev(np.ones((1, 100), np.float32))
    s = _stream(100, 2, payload, table)
    with pytest.raises(pmsz.PmszError) as e:
        pmsz.decode_edits(fhat, torch.from_numpy(np.frombuffer(s, np.uint8).copy()).cuda())
    assert e.value.status == 1


def test_valid_oddities_are_accepted():
    """A padded varint, bytes after the last entry, a chunk that starts late."""
    one = np.float32(1)
    for payload, table in ((b"\x80\x00\x81\x80\x00\x02\x01", None), (b"\x00\x01\x02\x01\xff\xff", None),
                           (b"\xff\x80\x00\x01\x02\x01", [(2, (1 << 64) - 1)])):
        s = _stream(100, 2, payload, table)
        g = host(pmsz.decode_edits(dev(np.ones((1, 100), np.float32)),
                                   torch.from_numpy(np.frombuffer(s, np.uint8).copy()).cuda()))
        want = np.ones((1, 100), np.float32)
        want[0, 0] = want[0, 3] = np.nextafter(one, np.float32(0))
        assert np.array_equal(g, want)


def test_malformed_payload_is_read_a_chunk_at_most():
    """No chunk reads past the bytes its entries can take: 2048 chunks of a 64 MiB
    payload in which no varint ends (a block that read on to the end of the
    payload would make 128 GiB of it, more than 15 ms at any rate of the memory)."""
    chunks, n = 2048, 2048 * 4096
    head = torch.from_numpy(np.frombuffer(_stream(n, n, b""), np.uint8).copy()).cuda()
    payload = torch.full((1 << 26,), 0x80, dtype=torch.uint8, device="cuda")
    head[24:32] = torch.tensor(list(struct.pack("<Q", payload.numel())), dtype=torch.uint8)
    fhat, s = torch.ones((1, n), device="cuda"), torch.cat([head, payload])
    assert s.numel() == 40 + 16 * chunks + payload.numel()
    ms = []
    for _ in range(3):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        with pytest.raises(pmsz.PmszError) as e:
            pmsz.decode_edits(fhat, s)
        t1.record()
        torch.cuda.synchronize()
        assert e.value.status == 1
        ms.append(t0.elapsed_time(t1))
    assert min(ms) < 5.0, ms
