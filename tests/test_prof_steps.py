"""The step table of a traced benchmark run finds each kernel under the name
that its launch shape and generator give it, whatever form of the generator's
step the call took."""
import json
import sqlite3


def test_step_table_takes_every_form_of_a_step(tmp_path):
    from paper_1101_1846_amd import prof  # not at collection: torch loads its HIP runtime first
    db, line = str(tmp_path / "run.db"), str(tmp_path / "line.json")
    con = sqlite3.connect(db)
    con.execute("create table kernels (name text, start integer, duration integer)")
    name = "void rngx::k_generate<rngx::%s, %d, 128, %d, 128, 2>(rngx::GenArgs)"
    t = 0
    # a tuning launch of the other form first, then the timed steps, then the fill and what comes after it
    for gen, dt, unroll, ns in ([("GenKISS", 1, 8, 900000)] + [("GenKISSMad", 1, 8, 200000 + i) for i in range(5)]
                                + [("GenXS256", 0, 4, 210000)] * 3):
        con.execute("insert into kernels values (?, ?, ?)", (name % (gen, dt, unroll), t, ns))
        t += 1
    con.execute("insert into kernels values ('at::native::FillFunctor<int>', ?, 1)", (t,))
    con.execute("insert into kernels values (?, ?, 5000000)", (name % ("GenKISS", 1, 8), t + 1))
    con.commit()
    con.close()
    with open(line, "w") as f:
        json.dump({"steps": 3, "roofline": {"kernel": "k_generate<KISS_f32> (store mode)", "avg_launch_ms": 0.2},
                   "launch_shapes": {"KISS_f32": {"wg": 128, "unroll": 8}, "XS256_u32": {"wg": 128, "unroll": 4}},
                   "per_kernel": {"KISS_f32": {"ms": 0.21}, "XS256_u32": {"ms": 0.22}}}, f)
    rows = prof.step_table(db, line).splitlines()[2:]
    assert rows[0] == "| k_generate<GenKISSMad, 1, 128, 8, 128, 2> | 3 | 200.00 | 200.00 | 200.00 | " \
                      "210.00 (timed steps: 200.00) |"
    assert rows[1] == "| k_generate<GenXS256, 0, 128, 4, 128, 2> | 3 | 210.00 | 210.00 | 210.00 | 220.00 |"
