"""Domains and boxes that run the box kernel: test_launch_plan.py holds the plan
to it on the host, test_gpu_box_runs.py compares the results."""

# (storage, ncomp, c_ns, forcing): the largest domains that take a box, deep and
# one plane, and boxes of uneven sizes that fit the format's threads
CASES = {
    ("f64", 2, 2, "shan-chen"): ([(45, 46, 47), (361, 363, 1)], [(9, 5, 3), (4, 3, 2), (1, 1, 1)]),
    ("f64", 2, 1, "guo"): ([(45, 46, 47), (361, 363, 1)], [(9, 5, 3), (7, 2, 5)]),
    ("f32", 2, 1, "guo"): ([(45, 46, 47), (361, 363, 1)], [(9, 5, 3), (4, 3, 2)]),
    ("f32", 2, 2, "shan-chen"): ([(57, 58, 59), (361, 363, 1)], [(13, 5, 3), (1, 1, 1)]),
    ("f16s", 2, 1, "shan-chen"): ([(63, 64, 65), (361, 363, 1)], [(13, 5, 3), (20, 4, 4)]),
    ("bf16s", 2, 2, "guo"): ([(63, 64, 65), (361, 363, 1)], [(13, 5, 3), (8, 4, 4)]),
    ("f64", 1, 1, "shan-chen"): ([(80, 81, 80), (361, 363, 1)], [(37, 5, 4), (1, 1, 1)]),
    ("f32", 1, 1, "guo"): ([(80, 81, 80), (361, 363, 1)], [(37, 5, 4), (13, 7, 9)]),
    ("f16s", 1, 1, "shan-chen"): ([(80, 81, 80), (361, 363, 1)], [(37, 5, 4), (4, 3, 2)]),
}

# the domain of the given boxes
BOXED = (37, 14, 9)
