"""Host logic of bench.py, on the CPU: the byte model of the operator's five passes and of a batch of
explicit steps, which the reported rates divide by, and the stored counter traffic of the stress
pass, reported only for the kernel sources it was taken on."""
import bench

VOXELS_256 = 256 ** 3


def test_operator_pass_bytes():
    # D_x p, five derivatives and p in, five stresses and Q out: 8 + 8 fields and the grain id
    assert bench.moved_bytes_per_voxel("x_sigma", 4) == 16 * 4 + 2
    assert bench.moved_bytes_per_voxel("x_sigma", 8) == 16 * 8 + 2
    # the whole apply: 47 fields and one grain id
    assert sum(bench.PASS_FIELDS.values()) == 47
    for real in (4, 8):
        assert sum(bench.moved_bytes_per_voxel(k, real) for k in bench.PASS_FIELDS) == 47 * real + 2


def test_explicit_batch_bytes():
    # one step: first pass 18, middle 32, last 15 fields; the grain id in two passes
    assert bench.explicit_bytes_per_voxel(1) == 65 * 8 + 4
    # a long batch: 53 fields, two grain ids and the mask a step
    assert abs(bench.explicit_bytes_per_voxel(10 ** 6) - (53 * 8 + 5)) < 1e-3
    assert bench.explicit_bytes_per_voxel(50) * 50 == (53 * 50 + 12) * 8 + 4 * 50 + 49


def test_stress_pass_counters(monkeypatch):
    for label, real in (("fp32", 4), ("fp64", 8)):
        t = bench.pmc_traffic("x_sigma", label, 256)
        if bench.sources_sha16() == bench.X_SIGMA_SOURCES:
            # FP64 reads p twice, the second time from the L2 but for 2% of it
            assert abs(t / (bench.moved_bytes_per_voxel("x_sigma", real) * VOXELS_256) - 1.0) < 0.02
        else:
            assert t is None
        assert bench.pmc_traffic("x_sigma", label, 512) is None
    monkeypatch.setattr(bench, "sources_sha16", lambda: "0" * 16)
    assert bench.pmc_traffic("x_sigma", "fp64", 256) is None
