"""The records that the device hands to the host, on the host-only runtime of
hip_stub.c: what a call allocates, what it does without, and whose slot it
writes."""
from hip_stub import run

COMMON = '''
out = (C.c_double * 4)()
def new(nx=64, ny=48):
    return ready(lattice(nx, ny), nx, ny)

def observe(h):
    return L.vanse_observe(h, out, None)
'''


def test_the_observables_without_allocation_allocate_nothing(tmp_path):
    run(tmp_path, COMMON + '''
fail_call = lambda name, k: name == "hipHostMalloc"   # so that no page is there yet
h = new()
fail_call = lambda name, k: 0
for _ in range(3):
    V.check(L.vanse_observe_noalloc(h, out, None))
assert "hipHostMalloc" not in calls and "hipHostFree" not in calls, calls
V.check(observe(h))                                    # this one may
assert calls.count("hipHostMalloc") == 1
del calls[:]
V.check(L.vanse_observe_noalloc(h, out, None))         # and now there is a slot
assert calls == ["hipStreamSynchronize"], calls
''')


def test_calls_succeed_without_pinned_memory(tmp_path):
    """No page (its allocation fails): the record is copied from the device."""
    run(tmp_path, COMMON + '''
fail_call = lambda name, k: name == "hipHostMalloc"
h = new()
V.check(L.vanse_set_void_fraction(h, field(64 * 48), None))
V.check(observe(h))
V.check(L.vanse_residual(h, out, None))
assert calls.count("hipHostMalloc") == 3 and calls.count("hipMemcpyAsync") == 3 + 1, calls
# a flag that the device sets there refuses the field
def launch(name, k):
    if "upload_fields" in name:
        C.c_int.from_address(C.c_void_p.from_address(launches[-1][2][5]).value).value = 1
    return 0
fail_launch = launch
assert L.vanse_set_void_fraction(h, field(64 * 48), None) == -1
''')


def test_more_calls_than_slots_at_once(tmp_path):
    """Seventy calls inside one another, each while the one before it waits:
    one allocation, no release, and no two with the same slot."""
    run(tmp_path, COMMON + '''
h = [new() for _ in range(70)]
depth, at, most, slots = 0, [], 0, []

def launch(name, k):
    if "reduce_partials" in name:
        slots.append(C.c_void_p.from_address(launches[-1][2][3]).value)
    return 0

def call(name, k):
    global depth
    if name == "hipStreamSynchronize" and depth < 70:
        d, depth = depth, depth + 1
        if depth < 70:
            V.check(observe(h[depth]))
    return 0

V.check(observe(h[0]))
del calls[:]
fail_launch, fail_call = launch, call
V.check(observe(h[0]))
assert len(slots) == 70 and len(set(slots)) == 70
assert "hipHostMalloc" not in calls and "hipHostFree" not in calls
''')


def test_a_slot_that_may_still_be_written_is_not_leased_again(tmp_path):
    run(tmp_path, COMMON + '''
h = new()
slots = []
def launch(name, k):
    if "upload_fields" in name:
        slots.append(C.c_void_p.from_address(launches[-1][2][5]).value)
    return 0
fail_launch = launch
fail_call = lambda name, k: name == "hipStreamSynchronize"
assert L.vanse_set_void_fraction(h, field(64 * 48), None) == -3
stub.hipGetLastError()
fail_call = lambda name, k: 0
V.check(L.vanse_set_void_fraction(h, field(64 * 48), None))
V.check(L.vanse_set_void_fraction(h, field(64 * 48), None))
assert slots[1] != slots[0] and slots[2] == slots[1], slots
# all lost: calls go on, by copies
fail_call = lambda name, k: name == "hipStreamSynchronize"
for _ in range(70):
    assert L.vanse_set_void_fraction(h, field(64 * 48), None) == -3
    stub.hipGetLastError()
fail_call = lambda name, k: 0
V.check(L.vanse_set_void_fraction(h, field(64 * 48), None))
V.check(observe(h))
''')


def test_the_static_scratch_holds_every_lattice_that_the_call_takes(tmp_path):
    """The limit is 131072 blocks of 256 columns of a row; the records are one per
    workgroup of the read-out, most of them on two rows."""
    run(tmp_path, COMMON + '''
size = C.c_size_t.in_dll(stub, "stub_var_bytes").value
for nx, ny in ((65536 * 256, 2), (254 * 2049, 3), (254 * 1900, 9), (512, 4099), (2, 65535)):
    h = ready(lattice(nx, ny, "f16s"), nx, ny)
    V.check(L.vanse_observe_noalloc(h, out, None))
    blocks = [b for name, b, _ in launches if "read_out" in name]
    assert len(blocks) == 1 and (blocks[0] + 1025) * 40 <= size, (nx, ny, blocks, size)
    L.vanse_destroy(h)
    keep.clear()
h = lattice(65536 * 256 + 1, 2, "f16s")
assert L.vanse_observe_noalloc(h, out, None) == -1
assert size < 3e6
''')
