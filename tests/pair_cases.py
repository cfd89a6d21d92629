"""Runs and groups whose default schedule takes two-step passes, for the tests that need them to."""
from paper_2504_20169_amd import lbm
from paper_2504_20169_amd import workloads as wl

# (lattice, storage, nx, ny, edges along x, along y, PML width, options)
SINGLE = [
    (37, "f64", 691, 641, "nrbc", "nrbc", 5, {}),
    (37, "f64", 660, 659, "nrbc", "nrbc", 4, dict(outlet="nrbc_a")),
    (37, "f64", 660, 661, "nrbc", "nrbc", 4, dict(terms=7)),
    (37, "f64", 4500, 103, "zg", "periodic", 20, {}),      # 97 interior rows
    (37, "f64", 102, 4500, "periodic", "nrbc", 0, {}),     # 96 interior columns
    (37, "f64", 106, 4900, "nrbc", "zg", 0, {}),           # 96 interior columns off two rings
    (37, "f32", 1024, 903, "nrbc", "zg", 3, {}),
    (37, "f32", 1009, 1001, "nrbc", "periodic", 0, dict(outlet="nrbc_a")),
    (17, "f64", 661, 653, "nrbc", "nrbc", 3, dict(terms=2)),
    (17, "f32", 1001, 997, "periodic", "periodic", 0, {}),
    (9, "f64", 690, 671, "nrbc", "nrbc", 9, dict(terms=5)),
    (9, "f32", 1203, 909, "nrbc", "nrbc", 5, dict(outlet="nrbc_a")),
]

# members of a group that pairs: the first by itself, the others with it, down to 96 interior cells
# a side; and the steps that each is asked for
GROUP = [
    ((700, 650, "zg", "zg", 4, {}), 40),
    ((98, 104, "nrbc", "nrbc", 6, {}), 17),                # 96 interior columns
    ((161, 98, "periodic", "nrbc", 5, {}), 9),             # 96 interior rows
    ((109, 155, "zg", "periodic", 1, {}), 40),
    ((120, 131, "nrbc", "nrbc", 8, dict(outlet="nrbc_a")), 16),
    ((113, 99, "nrbc", "nrbc", 7, dict(terms=2)), 0),
    ((102, 102, "periodic", "periodic", 0, {}), 1),
]


def make(lattice, storage, nx, ny, bcx, bcy, W, kw, seed, overlap=2):
    r = lbm.Run(nx, ny, 0.8, 1.0, 0.05, 0.01, 1.0, storage=storage, lattice=lattice)
    r.set_bc(lbm.LBM_XMIN | lbm.LBM_XMAX, bcx)
    r.set_bc(lbm.LBM_YMIN | lbm.LBM_YMAX, bcy)
    if "outlet" in kw:
        r.set_bc(lbm.LBM_XMAX, kw["outlet"])
    mask = (3 if bcx != "periodic" else 0) | (12 if bcy != "periodic" else 0)
    if W and mask:
        r.set_pml(mask, W, 0.002)
    if "terms" in kw:
        r.set_nrbc_pml_terms(kw["terms"])
    r.set_launch(overlap=overlap)
    Nx, Ny = r.grid()
    r.init(*wl.noisy_state(Nx, Ny, seed, 1.0, 0.05, 0.01, 1.0).as_tuple())
    return r
