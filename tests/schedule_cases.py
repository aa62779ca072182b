"""Shapes whose calls without a plan run on the tiles that no plan names, and
the library's choice for them."""
from paper_2607_12505_amd import nmspmm
from paper_2607_12505_amd.nmprobe import schedule_tile  # noqa: F401

PATTERN = {nmspmm.NM_KIND_SP42: (2, 4), nmspmm.NM_KIND_C14: (1, 4), nmspmm.NM_KIND_C28: (2, 8),
           nmspmm.NM_KIND_MK4: (4, 8), nmspmm.NM_KIND_DENSE: (8, 8)}

# (m, n, k, kind, outputs, tile): ragged tokens, channels that are no multiple
# of 16 (a partial last fragment and 16-byte chunk), reductions that are no
# multiple of 128; one to three k-steps on the wide tiles (test_gpu_schedule.py
# runs every tile past its ring), up to twelve on the others
CASES = [
    (3674, 2524, 128, nmspmm.NM_KIND_SP42, nmspmm.NM_OUT_I8, 12),
    (4142, 1996, 144, nmspmm.NM_KIND_SP42, nmspmm.NM_OUT_F16, 12),
    (2758, 3116, 272, nmspmm.NM_KIND_DENSE, nmspmm.NM_OUT_F16, 12),
    (5472, 1792, 272, nmspmm.NM_KIND_C14, nmspmm.NM_OUT_I8, 12),
    (3094, 2656, 144, nmspmm.NM_KIND_MK4, nmspmm.NM_OUT_F16, 12),
    (5447, 152, 1040, nmspmm.NM_KIND_SP42, nmspmm.NM_OUT_I32, 13),
    (5741, 136, 1504, nmspmm.NM_KIND_DENSE, nmspmm.NM_OUT_I8, 13),
    (4218, 388, 976, nmspmm.NM_KIND_SP42, nmspmm.NM_OUT_F16, 14),
    (2941, 660, 368, nmspmm.NM_KIND_DENSE, nmspmm.NM_OUT_F16, 14),
    (1817, 1032, 1200, nmspmm.NM_KIND_C14, nmspmm.NM_OUT_I8, 14),
    (4621, 3344, 144, nmspmm.NM_KIND_SP42, nmspmm.NM_OUT_I8, 15),
    (5147, 3216, 144, nmspmm.NM_KIND_DENSE, nmspmm.NM_OUT_F16, 15),
    (5014, 3508, 128, nmspmm.NM_KIND_C28, nmspmm.NM_OUT_F16, 15),
    (5186, 3412, 128, nmspmm.NM_KIND_MK4, nmspmm.NM_OUT_F16, 15),
]
