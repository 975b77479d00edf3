"""Simulation set-up and stepping of liblpic.so on the host: its sequence of allocations and
launches under a stand-in HIP runtime (hip_host_stub.cpp) in a process of its own, where memory
can run out and a launch can fail at a chosen place without a GPU."""
import ctypes
import importlib.util
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2607_13507_amd")
NX, NY, SLOTS = 128, 64, 30000


def _child(case, tmp_path):
    so = str(tmp_path / "stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7",
                    "-o", so, os.path.join(HERE, "hip_host_stub.cpp")], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), case, so], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


class Host:
    """The stand-in runtime, the library bound to it, and one 2D FP64 box (its arrays, too, come
    from the stand-in)."""

    def __init__(self, so):
        self.stub = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        for name, res, args in (("stub_used", ctypes.c_size_t, []),
                                ("stub_budget", None, [ctypes.c_size_t]),
                                ("stub_newest", ctypes.c_void_p, [ctypes.c_size_t]),
                                ("stub_events", ctypes.c_char_p, [])):
            f = getattr(self.stub, name)
            f.restype, f.argtypes = res, args
        spec = importlib.util.spec_from_file_location("lpic", os.path.join(PKG, "lpic.py"))
        self.L = L = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(L)
        lib = ctypes.CDLL(L.LIB_PATH)
        for name, (res, args) in L.EXPORTS.items():
            getattr(lib, name).restype, getattr(lib, name).argtypes = res, args
        L._lib = lib
        self.grid = L.Grid(2, NX, NY, 1, 0.1, 0.1, 1.0, 0.05, 0.0, 0, 0)
        self.fields = L.Fields(*[self.alloc(NX * NY * 8) for _ in range(11)])
        self.sp, self.alt = self.species(), self.species()

    def alloc(self, n):
        p = ctypes.c_void_p()
        assert self.stub.hipMalloc(ctypes.byref(p), ctypes.c_size_t(n)) == 0
        return p.value

    def species(self):
        a = [self.alloc(SLOTS * 8) for _ in range(6)]
        return self.L.Species(SLOTS, -1.0, 1.0, 2, 0, None, None, None, None, a[0], a[1], None,
                              *a[2:])

    def create(self, species=True, flags=0, diag=0, graph=True, open_x=False):
        L = self.L
        o = L.Options(L.Tiling(16, 16, 1, 5, 256, flags), 10, diag, int(graph), 0)
        self.grid.open_x = int(open_x)
        sp, alt = ([self.sp], [self.alt]) if species else ([], [])
        return L.lpic_sim_create([self.grid], [self.fields], sp, [0] * len(sp), alt, L.F64_ABS, o,
                                 0)

    def tile(self, h):
        t = self.L.lpic_get_stats(h).field_tile
        return t[0], t[1]

    def events(self):
        return self.stub.stub_events().decode().splitlines()

    def kernels(self):
        """Names of the launched kernels (template arguments left out), in order."""
        out = []
        for e in self.events():
            if e.startswith("launch "):
                name = e.split()[1]
                out.append(name[name.index("k_"):].split("I")[0])
        return out


# ---- the cases, each in a process of its own -------------------------------------------------
def memory(H):
    """The second field set takes what the required buffers leave: not created before them, and
    given back when one that is needed later finds no room."""
    set2 = 9 * NX * NY * 8
    u0 = H.stub.stub_used()
    for flags in (0, H.L.ESCAPE_REBIN):
        h = H.create(flags=flags | H.L.FIELD_SEPARATE)
        need = H.stub.stub_used() - u0
        H.L.lpic_sim_destroy(h)
        # room for the required memory and all but one byte of the set
        H.stub.stub_budget(u0 + need + set2 - 1)
        h = H.create(flags=flags)
        assert H.tile(h) == (0, 0)
        H.L.lpic_step(h, 3)
        assert "k_yee_mid" not in H.kernels()
        H.L.lpic_sim_destroy(h)
        H.stub.stub_budget(2 ** 63)
        h = H.create(flags=flags)
        assert H.tile(h) == (64, 16)
        H.kernels()
        H.L.lpic_step(h, 3)
        assert H.kernels().count("k_yee_mid") == 2
        # the split path's buffer: room only where the set is
        H.stub.stub_budget(H.stub.stub_used())
        hook = H.L.HOOK_FN(lambda *_: 0)
        H.L.lpic_register_hook(h, H.L.STAGE["INTERPOLATOR"], hook, None)
        H.L.lpic_step(h, 2)
        assert H.tile(h) == (0, 0)
        H.L.lpic_clear_hooks(h)
        H.L.lpic_step(h, 3)
        assert "k_yee_mid" not in H.kernels()
        H.L.lpic_sim_destroy(h)
        H.stub.stub_budget(2 ** 63)
        assert H.stub.stub_used() == u0


def layers(H):
    """PML layers that find no room beside the set."""
    h = H.create(species=False, open_x=True)
    assert H.tile(h) == (64, 16)
    H.stub.stub_budget(H.stub.stub_used())
    H.L.lpic_set_pml(h, 0, H.L.Pml(8, 3, 1, 0, -1.0, 1.0, 0.0))
    H.L.lpic_step(h, 3)
    assert "k_pml" not in H.kernels()


def unused(H):
    """No second set where no step can use it, and none left over from before."""
    u0 = H.stub.stub_used()
    h = H.create(species=False, flags=H.L.FIELD_SEPARATE)
    need = H.stub.stub_used() - u0
    H.L.lpic_sim_destroy(h)
    h = H.create(species=False, diag=1)
    assert H.tile(h) == (64, 16)
    assert H.stub.stub_used() - u0 == need
    H.L.lpic_step(h, 3)
    assert "k_yee_mid" not in H.kernels()
    for diag, flags, fused in ((4, 0, True), (4, H.L.FIELD_SEPARATE, False), (1, 0, False)):
        H.L.lpic_set_options(h, H.L.Options(H.L.Tiling(16, 16, 1, 5, 256, flags), 10, diag, 1, 0))
        assert (H.stub.stub_used() - u0 > need) == fused, (diag, flags)
        H.L.lpic_step(h, 3)
        assert ("k_yee_mid" in H.kernels()) == fused, (diag, flags)


def clears(H):
    """What set-up clears on the null stream is there before a call returns: the caller's stream
    may be one that does not wait for the null stream."""
    def last_clear_is_waited_for():
        e = H.events()
        last = max((i for i, x in enumerate(e) if x == "memset"), default=-1)
        return last >= 0 and any(x.startswith("wait") for x in e[last + 1:])
    for species in (False, True):
        for flags in (0, H.L.FIELD_SEPARATE, H.L.ESCAPE_REBIN):
            H.events()
            h = H.create(species=species, flags=flags, open_x=True)
            assert last_clear_is_waited_for(), (species, flags)
            H.L.lpic_set_laser(h, 0, H.L.Laser(1, 4, 1.0, 1.0, 1.0, 3.0, 0.0, 0.0, 10.0))
            assert last_clear_is_waited_for(), (species, flags)
            H.L.lpic_set_pml(h, 0, H.L.Pml(8, 3, 1, 0, -1.0, 1.0, 0.0))
            assert last_clear_is_waited_for(), (species, flags)
            H.L.lpic_sim_destroy(h)


def second_set_current(H):
    """Only a box without species has its second J cleared at set-up (nothing else does it)."""
    set2 = 9 * NX * NY * 8
    for species in (False, True):
        h = H.create(species=species)
        p = H.stub.stub_newest(set2)
        ctypes.memset(p, 7, set2)
        H.L.lpic_set_laser(h, 0, None)                   # reconfigures, keeps the set
        assert H.stub.stub_newest(set2) == p
        a = ctypes.string_at(p, set2)
        assert a[:set2 // 3 * 2] == b"\7" * (set2 // 3 * 2)
        assert a[set2 // 3 * 2:] == (b"\7" if species else b"\0") * (set2 // 3)
        H.L.lpic_sim_destroy(h)


def failed_call(H):
    """An error in the middle of a call whose fields are in the second set brings them back to
    the caller's arrays, with their half of psi and their clock word."""
    n = NX * NY * 8
    cells = 8
    psi = 2 * 4 * NY * 2 * cells * 8                      # two halves, a coefficient table after
    table = 2 * 2 * cells * 3 * 8
    for graph, steps, fail in ((True, 3, "instantiate"), (False, 3, "launch"), (False, 2, "launch")):
        h = H.create(species=graph, graph=graph, open_x=True)
        H.L.lpic_set_laser(h, 0, H.L.Laser(1, 12, 1.0, 1.0, 1.0, 3.0, 0.0, 0.0, 10.0))
        H.L.lpic_set_pml(h, 0, H.L.Pml(cells, 3, 1, 0, -1.0, 1.0, 0.0))
        H.L.lpic_step(h, 1)                               # (the first sort is not captured)
        H.events()
        p = H.stub.stub_newest(9 * n)
        q = H.stub.stub_newest(psi + table)
        arrays = [getattr(H.fields, k) for k, _ in H.L.Fields._fields_[:9]]
        for k in range(9):
            ctypes.memset(arrays[k], 0, n)
            ctypes.memset(p + k * n, k + 1, n)
        ctypes.memset(q, 0, psi // 2)
        ctypes.memset(q + psi // 2, 5, psi // 2)
        if fail == "instantiate":
            H.stub.stub_fail_instantiate(1)               # the second step's variant
        else:                                             # the third launch: the fields have moved
            H.stub.stub_fail_launch(3 if steps == 3 else 2)
        try:
            H.L.lpic_step(h, steps)
            raise AssertionError("no error")
        except H.L.LpicError as e:
            assert e.status == -2 and "stub error" in str(e), e
        assert H.events().count("copy") == 11
        for k in range(9):
            assert ctypes.string_at(arrays[k], n) == bytes([k + 1]) * n, (graph, steps, k)
        assert ctypes.string_at(q, psi // 2) == b"\5" * (psi // 2)
        H.L.lpic_step(h, 3)                               # and the simulation goes on
        # nothing to bring back before the first move is complete
        if not graph:
            H.stub.stub_fail_launch(1)
            try:
                H.L.lpic_step(h, 2)
                raise AssertionError("no error")
            except H.L.LpicError:
                pass
            assert "copy" not in H.events()
            # fields that cannot be brought back: later calls are refused
            H.stub.stub_fail_launch(2)
            H.stub.stub_fail_copy(4)
            for text in ("stub error", "lost"):
                try:
                    H.L.lpic_step(h, 2)
                    raise AssertionError("no error")
                except H.L.LpicError as e:
                    assert e.status == -2 and text in str(e), e
        H.L.lpic_sim_destroy(h)


def rebinned(H):
    """The two escape lists of a re-binned step are short or empty: no deposit boxes in LDS."""
    h = H.create(flags=H.L.ESCAPE_REBIN)
    H.L.lpic_step(h, 2)
    e = [x.split() for x in H.events() if "k_escape" in x]
    assert len(e) == 4
    assert all(x[3] == "0" for x in e), e


def moved_window(H):
    """A simulation whose window has moved keeps the fused field update, with the same tile
    before and after its options are set again."""
    H.grid.nx, H.grid.ny = 96, 24
    h = H.create(open_x=True)

    def updates():
        H.L.lpic_step(h, 3)
        return [e for e in H.events() if "k_yee_mid" in e]
    first = updates()
    assert len(first) == 2 and H.tile(h) == (32, 8)
    H.L.lpic_window_shift(h, 0, 5)
    assert updates() == first
    H.L.lpic_set_options(h, H.L.Options(H.L.Tiling(16, 16, 1, 5, 256, 0), 10, 0, 1, 0))
    assert updates() == first


# ---- the tests -------------------------------------------------------------------------------
def test_required_memory_before_the_second_field_set(tmp_path):
    _child("memory", tmp_path)


def test_layers_before_the_second_field_set(tmp_path):
    _child("layers", tmp_path)


def test_no_second_field_set_where_none_is_used(tmp_path):
    _child("unused", tmp_path)


def test_clears_are_done_when_a_call_returns(tmp_path):
    _child("clears", tmp_path)


def test_current_of_the_second_field_set(tmp_path):
    _child("second_set_current", tmp_path)


def test_error_in_the_middle_of_a_call(tmp_path):
    _child("failed_call", tmp_path)


def test_escape_launches_of_a_rebinned_step(tmp_path):
    _child("rebinned", tmp_path)


def test_fused_update_of_a_moved_window(tmp_path):
    _child("moved_window", tmp_path)


if __name__ == "__main__":
    globals()[sys.argv[1]](Host(sys.argv[2]))
