"""Measurement studies beside bench.py: each prints one JSON line per case.

  python studies.py size   [--steps 200]   # single-Block periodic cubes
  python studies.py blocks [--steps 200]   # 384^3 split into 1..216 Blocks, porous
  python studies.py open   [--steps 200]   # open x faces against periodic x
  python studies.py pad    [--steps 200]   # odd Block sizes and row padding
  python studies.py hbm                    # HBM ceilings of plain access patterns
  python studies.py hetero [--steps 50]    # host-CPU Blocks next to the GPU's
  python studies.py precision              # shifted FP16/BF16 against FP32/FP64 storage
  python studies.py warmstart              # learned warm start against a start from rest
  python studies.py conv                   # per-layer times of the convolution kernels
  python studies.py persistent             # graph-launched steps against the persistent sweep

size:   periodic cube N^3 (N = 64..512 step 32) as one Block, FP32 and FP64
        storage, started from rest with g_x = 1e-6, tau 0.8: MLUPS against N,
        the single-Block scaling study of Sec. 5.1.
blocks: the 384^3 periodic cube as 1, 8, 27, 64 and 216 equal Blocks, and
        the 512x256x256 porous channel as its uneven Blocks; per-launch times
        of the sweep and of the separate ghost exchange (HIP events) for the
        three exchange schedules (0 copy kernel, 2 x faces written by the
        sweep, 1 fully fused), for the porous channel in its uneven Blocks and
        for 64 uneven Blocks (4x4x4, edges from {32, 48, 64}): the cost of
        Blocks and of their on-GPU copies, Sec. 5.1.
pad:    single-Block periodic cubes of odd and even edge around 64, 70,
        128 and 256 (the paper's odd-size effects, Sec. 5.1) with rows
        aligned to 128-byte lines and no extra padding (row_pad -1) or one
        or two extra lines per row, with streaming stores, and without
        padding with ordinary stores, FP32 and FP64: MLUPS against the edge.
hbm:    over 2 GiB buffers (well past the 256 MB Infinity Cache): read-only,
        write-only and copy streams (grid-strided, and one contiguous chunk
        per workgroup), a two-read one-write triad, the sweep's 19-read
        19-write stream pattern without arithmetic, with 1-8 accesses in
        flight per thread, streaming or ordinary, several grid sizes; and the
        runtime's device-to-device copy and fill: the attainable bandwidth of
        each pattern (lbm_hbm_probe), against which the sweep (one read and
        one write of every value, the copy pattern) is read.
hetero: the porous 512x256x256 channel in its uneven Blocks, FP32 (Sec. 5.3's
        heterogeneous study on one node): the GPU alone, then the last k
        Blocks on the host CPU (k = 1, 2, 4, 8, 16, 16 threads) with the GPU
        sweep, host sweep, exchange and whole-step times of phase-timed steps
        and the step time of lbm_step's pipelined steps; the host sweep's
        rate against its thread count on the last Block; and the static load
        balance (lbm_balance_host_blocks).
open:   a 512x256x256 duct (y periodic, z walls), FP32: x periodic with a
        body force against a velocity inlet and a pressure outlet on the x
        faces, as one Block, 4 Blocks along x, 4x2x2 Blocks and the porous
        channel's uneven Blocks; the second column of times is then the
        post-sweep work (exchange and the boundary nodes of the open faces).
precision: the n^3 lid-driven cavity (tau 0.55, lid 0.1 on +z, 5000 steps)
        in every storage precision: MLUPS, the speedup of shifted FP16/BF16
        storage over FP32, and the normwise velocity error of each run against
        the GPU FP64 run of the same size (the 96^3 instance against the CPU
        oracle is a GPU test, tests/test_gpu_precision.py).
warmstart: the learned warm start of the 64x64x128 porous channels: N training
        steady states generated by the solver, the U-Net trained on them, and
        M held-out seeds run from rest and from the prediction against a
        tightly converged FP64 reference: steps and wall-clock time to the
        residual criterion and to velocity errors of 1e-2 ... 3e-4.
conv:   per-layer times of the three convolution kernels of the U-Net at
        batch 8, 64x64x128 (HIP events): TFLOP/s against the BF16 MFMA peak.
persistent: microseconds per step of graph-launched steps (10 and 50 per
        graph) against the persistent multi-step sweep (100 and 1000 steps per
        launch) on the 32^3 cavity, a 64x64x128 porous channel, 128^3 as one
        and as eight Blocks, and the 256^3 channel.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

from paper_1007_1388_amd import inputs, lbm  # noqa: E402

HBM_PEAK_GBS = 8000.0


def measure(dims, precision, steps, blocks=None, solid=None, walls=(False, False, False), tau=0.8,
            force=(1e-6, 0.0, 0.0), fused=0, graph_steps=10, open_x=None, row_pad=0, nontemporal=None):
    """nontemporal None: the library's default for the grid."""
    import torch
    lat = lbm.Lattice(dims, blocks=blocks, walls=walls, tau=tau, force=force, precision=precision,
                      open_faces=open_x, row_pad=row_pad)
    if solid is not None:
        lat.set_geometry(solid)
    sch = dict(fused_exchange=fused, graph_steps=graph_steps)
    if nontemporal is not None:
        sch["nontemporal"] = nontemporal
    lat.set_schedule(**sch)
    lat.step(20)
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    lat.step(steps)
    e1.record()
    torch.cuda.synchronize()
    step_ms = e0.elapsed_time(e1) / steps
    sweep_ms, exch_ms = lat.step_timed(min(steps, 100))
    info = lat.info()
    lat.sums()
    lat.close()
    nf = info["n_fluid"]
    return dict(step_ms=round(step_ms, 5), sweep_ms=round(sweep_ms, 5), exchange_ms=round(exch_ms, 5),
                mlups=round(nf / step_ms / 1e3, 1),
                sweep_gbs=round(nf * info["bytes_per_update"] / (sweep_ms * 1e-3) / 1e9, 1),
                frac=round(nf * info["bytes_per_update"] / (sweep_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
                blocks=info["n_blocks"], fluid_cells=nf)


def size_sweep(steps, sizes):
    for n in sizes:
        for prec in ("f32", "f64"):
            try:
                r = measure((n, n, n), prec, steps)
            except lbm.LBMError as e:  # one Block beyond the size limit
                print(json.dumps(dict(study="size", n=n, precision=prec, refused=str(e))), flush=True)
                continue
            print(json.dumps(dict(study="size", n=n, precision=prec, **r)), flush=True)


def block_sweep(steps):
    n = 384
    for k in (1, 2, 3, 4, 6):
        blocks = inputs.uniform_blocks((n, n, n), (k, k, k))
        for fused in (0, 2, 1):
            r = measure((n, n, n), "f32", steps, blocks=blocks, fused=fused)
            print(json.dumps(dict(study="blocks", domain="384^3 periodic", split="%dx%dx%d" % (k, k, k),
                                  precision="f32", fused=fused, **r)), flush=True)
    p = inputs.preset("porous512")
    blocks = inputs.uneven_blocks(p["dims"], p["block_edges"], seed=0)
    solid = inputs.porous_spheres(p["dims"], p["solid_fraction"], p["radius"], seed=0)
    for fused in (0, 2, 1):
        r = measure(p["dims"], "f32", steps, blocks=blocks, solid=solid, walls=p["walls"], tau=p["tau"],
                    force=p["force"], fused=fused)
        print(json.dumps(dict(study="blocks", domain="porous 512x256x256", split="uneven {32,48,64}",
                              precision="f32", fused=fused, **r)), flush=True)
    # the literal 64 uneven Blocks: a 4x4x4 grid with edges from {32, 48, 64},
    # the domain being whatever the edges sum to
    dims, blocks = inputs.uneven_blocks_grid((4, 4, 4), p["block_edges"], seed=0)
    solid = inputs.porous_spheres(dims, p["solid_fraction"], p["radius"], seed=0)
    for fused in (0, 2, 1):
        r = measure(dims, "f32", steps, blocks=blocks, solid=solid, walls=p["walls"], tau=p["tau"],
                    force=p["force"], fused=fused)
        print(json.dumps(dict(study="blocks", domain="porous %s" % "x".join(map(str, dims)),
                              split="4x4x4 uneven {32,48,64}", precision="f32", fused=fused, **r)), flush=True)


def pad_sweep(steps):
    for n in (63, 64, 65, 69, 70, 71, 72, 127, 128, 129, 255, 256, 257):
        for prec in ("f32", "f64"):
            for rp, nt in ((-1, 1), (1, 1), (2, 1), (-1, 0)):
                r = measure((n, n, n), prec, steps, row_pad=rp, nontemporal=nt)
                print(json.dumps(dict(study="pad", n=n, precision=prec, row_pad=rp, nontemporal=nt, **r)),
                      flush=True)


def hbm_moved(kind, nbytes):
    """Bytes one pass of lbm_hbm_probe kind moves over `nbytes` buffers."""
    if kind in (0, 1, 7):
        return nbytes
    if kind == 4:
        return 3 * nbytes
    if kind == 5:
        per = nbytes // 19 // 4096 * 4096
        while 19 * per + 18 * 768 > nbytes:
            per -= 4096
        return 2 * 19 * per
    return 2 * nbytes


HBM_KINDS = {0: "read", 1: "write", 2: "copy", 3: "copy, one chunk per workgroup", 4: "triad 2 reads 1 write",
             5: "19-stream sweep pattern", 6: "hipMemcpy device to device", 7: "hipMemset"}


def hbm_sweep(reps=10):
    import torch
    nbytes = 2 << 30
    a = torch.ones(nbytes // 2, dtype=torch.float32, device="cuda")   # two buffers of nbytes (the triad's)
    b = torch.zeros(nbytes // 4, dtype=torch.float32, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    for kind in (0, 1, 2, 3, 4, 5, 6, 7):
        unrolls = (1,) if kind in (6, 7) else ((1, 2, 4) if kind == 5 else (1, 2, 4, 8))
        grids = (0,) if kind in (6, 7) else (256, 512, 1024, 4096, 16384, 65536)
        for unroll in unrolls:
            for nt in ((1,) if kind in (6, 7) else (1, 0)):
                for grid in grids:
                    ms = lbm.lbm_hbm_probe(kind, unroll, nt, a.data_ptr(), b.data_ptr(), nbytes, grid, reps, st)
                    gbs = hbm_moved(kind, nbytes) / (ms * 1e-3) / 1e9
                    print(json.dumps(dict(study="hbm", pattern=HBM_KINDS[kind], kind=kind, unroll=unroll,
                                          nontemporal=nt, grid=grid, ms=round(ms, 5), gbs=round(gbs, 1),
                                          frac=round(gbs / HBM_PEAK_GBS, 4))), flush=True)


def hetero_sweep(steps, threads=16):
    import torch
    p = inputs.preset("porous512")
    blocks = inputs.uneven_blocks(p["dims"], p["block_edges"], seed=0)
    solid = inputs.porous_spheres(p["dims"], p["solid_fraction"], p["radius"], seed=0)
    lat = lbm.Lattice(p["dims"], blocks=blocks, walls=p["walls"], tau=p["tau"], force=p["force"], precision="f32")
    lat.set_geometry(solid)
    nb = len(blocks)
    nf = lat.info()["n_fluid"]
    lat.step(20)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    lat.step(steps)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    print(json.dumps(dict(study="hetero", case="gpu alone", blocks=nb, host_blocks=0, step_ms=round(ms, 4),
                          mlups=round(nf / ms / 1e3, 1))), flush=True)
    # host sweep rate against threads, last Block
    for th in (1, 2, 4, 8, 16):
        lat.set_host_blocks([nb - 1], threads=th)
        lat.step(2)
        g, c, x, s = lat.step_host_timed(max(5, steps // 5))
        fh = _fluid(solid, blocks[nb - 1:])
        print(json.dumps(dict(study="hetero", case="host rate", threads=th, host_fluid=fh, cpu_ms=round(c, 4),
                              host_mlups=round(fh / c / 1e3, 1))), flush=True)
    for k in (1, 2, 4, 8, 16):
        ids = list(range(nb - k, nb))
        lat.set_host_blocks(ids, threads=threads)
        lat.step(2)
        g, c, x, s = lat.step_host_timed(steps)
        # the same split stepped as lbm_step runs it (the next GPU sweep
        # queued behind the exchange)
        t0 = time.perf_counter()
        lat.step(steps)
        torch.cuda.synchronize()
        sp = (time.perf_counter() - t0) * 1e3 / steps
        fh = _fluid(solid, blocks[nb - k:])
        print(json.dumps(dict(study="hetero", case="split", threads=threads, host_blocks=k, host_fluid=fh,
                              gpu_sweep_ms=round(g, 4), cpu_sweep_ms=round(c, 4), exchange_ms=round(x, 4),
                              step_ms=round(s, 4), pipelined_step_ms=round(sp, 4),
                              mlups=round(nf / sp / 1e3, 1))), flush=True)
    lat.set_host_blocks([])
    k, tg, th = lat.balance_host_blocks(threads=threads, trial_steps=steps)
    print(json.dumps(dict(study="hetero", case="balance", threads=threads, host_blocks=k, gpu_alone_ms=round(tg, 4),
                          split_ms=round(th, 4))), flush=True)
    lat.close()


def _fluid(solid, blocks):
    n = 0
    for lo, hi in blocks:
        # solid is [z][y][x]
        n += int((solid[lo[2]:hi[2], lo[1]:hi[1], lo[0]:hi[0]] == 0).sum())
    return n


def open_sweep(steps):
    dims = (512, 256, 256)
    opn = {"-x": ("velocity", (0.02, 0.0, 0.0)), "+x": ("pressure", 1.0)}
    opy = {"-y": ("velocity", (0.0, 0.02, 0.0)), "+y": ("pressure", 1.0)}
    for label, walls, force, ox in (("x periodic, g_x = 1e-6", (False, False, True), (1e-6, 0, 0), None),
                                    ("x velocity inlet / pressure outlet", (True, False, True), (0, 0, 0), opn),
                                    ("y velocity inlet / pressure outlet (x periodic)", (False, True, True),
                                     (0, 0, 0), opy)):
        for split in ((1, 1, 1), (4, 1, 1), (4, 2, 2), "uneven"):
            if split == "uneven":
                blocks = inputs.uneven_blocks(dims, (32, 48, 64), seed=0)
                name = "uneven {32,48,64}"
            else:
                blocks = inputs.uniform_blocks(dims, split)
                name = "%dx%dx%d" % split
            for fused in ((0,) if split == (1, 1, 1) else (0, 2)):
                r = measure(dims, "f32", steps, blocks=blocks, walls=walls, force=force, fused=fused, open_x=ox)
                print(json.dumps(dict(study="open", domain="512x256x256 duct", x=label, split=name,
                                      precision="f32", fused=fused, **r)), flush=True)


PRECS = ["f64", "f32", "f16s", "bf16s"]


def precision_run(n, steps, prec, tau, lid):
    import numpy as np
    import torch
    lat = lbm.Lattice((n, n, n), walls=(True, True, True), wall_u={"+z": (lid, 0, 0)}, tau=tau, precision=prec)
    lat.set_schedule(graph_steps=10)
    lat.step(10)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    lat.step(steps - 10)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    sweep_ms, _ = lat.step_timed(50)
    info = lat.info()
    rho, u = lat.macroscopic()
    m, _ = lat.sums()
    lat.close()
    return dict(u=u, mlups=n ** 3 * (steps - 10) / dt / 1e6, seconds=dt, mass=m, sweep_ms=sweep_ms,
                frac=n ** 3 * info["bytes_per_update"] / (sweep_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                finite=bool(np.isfinite(m)))


def velocity_error(u, ref):
    import numpy as np
    d = u - ref
    return dict(linf=float(np.abs(d).max() / np.abs(ref).max()), l2=float(np.sqrt((d ** 2).sum() / (ref ** 2).sum())))


def precision_study(n=384, steps=5000, tau=0.55, lid=0.1):
    import numpy as np
    ref, f32 = None, None
    for p in PRECS:
        r = precision_run(n, steps, p, tau, lid)
        row = dict(study="precision", n=n, steps=steps, storage=p, mlups=round(r["mlups"], 1),
                   sweep_ms=round(r["sweep_ms"], 5), frac=round(r["frac"], 4), finite=r["finite"])
        if p == "f64":
            ref = r["u"]
        elif ref is not None and r["finite"]:
            row["err_vs_gpu_f64"] = velocity_error(r["u"], ref)
        if p == "f32":
            f32 = r["mlups"]
        elif p in ("f16s", "bf16s") and f32:
            row["speedup_vs_f32"] = round(r["mlups"] / f32, 3)
        row["umax"] = float(np.abs(r["u"]).max())
        print(json.dumps(row), flush=True)
        del r


# ---------------------------------------------------------------- warm start
TARGETS = (1e-2, 3e-3, 1e-3, 3e-4)


def ws_reference(gx, solid, tol=1e-10, max_steps=400_000):
    """Tightly converged steady velocity (device, FP64 storage): from rest to
    a two-step residual of `tol`, averaged over two consecutive steps (which
    removes any period-two part); returns (u, steps, residual)."""
    import torch
    from paper_1007_1388_amd import warmstart as ws
    lat = ws.make_lattice(gx, solid, None, precision="f64")
    (n, _, r), = ws.run_to_steady([lat], max_steps=max_steps, tol=tol)
    _, ua = lat.macroscopic_device()
    lat.step(1)
    _, ub = lat.macroscopic_device()
    torch.cuda.synchronize()
    lat.close()
    return 0.5 * (ua + ub), n, r


def ws_tracked(lat, u_ref, fluid, check_every=100, max_steps=60_000, steps0=0):
    """Steps to each accuracy target against u_ref (relative 2-norm over
    fluid cells) of the velocity itself and of its average over the last two
    steps, checked every `check_every` steps (a period-two oscillation that
    bounce-back sustains in some pore geometries, and that the two-step
    residual cannot see, shows only in the first).  Returns ({target: steps},
    {target: steps} of the average, final errors (velocity, average))."""
    import torch
    nref = torch.linalg.vector_norm(u_ref[:, fluid])
    hit, hit2, steps = {}, {}, steps0
    err = err2 = float("nan")
    while steps < max_steps:
        lat.step(check_every - 1)
        _, ua = lat.macroscopic_device()
        lat.step(1)
        _, u = lat.macroscopic_device()
        steps += check_every
        err = float(torch.linalg.vector_norm((u - u_ref)[:, fluid]) / nref)
        err2 = float(torch.linalg.vector_norm((0.5 * (u + ua) - u_ref)[:, fluid]) / nref)
        for tg in TARGETS:
            if tg not in hit and err < tg:
                hit[tg] = steps
            if tg not in hit2 and err2 < tg:
                hit2[tg] = steps
        if (len(hit) == len(TARGETS) and len(hit2) == len(TARGETS)) or not err2 < 1e30:
            break
    return hit, hit2, (err, err2)


def ws_evaluate(trainer, seeds, log=print):
    """Per held-out seed: steps and wall-clock time from rest and from the
    network's prediction (inference included) to the residual criterion,
    each a run of its own timed end to end; and, in further runs that read
    the velocity every 100 steps, the steps to each accuracy target against
    a tightly converged FP64 reference (their time is taken as steps times
    the wall-clock time per step of the timed run)."""
    import numpy as np
    import torch
    from paper_1007_1388_amd import warmstart as ws
    rows = []
    nx, ny, nz = ws.DIMS
    shape = (nz, ny, nx)
    for s in seeds:
        solid, gx, frac = ws.sample(s)
        d = dict(solid=torch.from_numpy(solid.reshape(-1)).cuda(), gx=gx)
        fluid = torch.from_numpy(solid == 0).cuda()
        u_ref, n_ref, r_ref = ws_reference(gx, solid)
        n0, secs0, _ = ws.solve(gx, solid)
        n1, secs1, _ = ws.solve(gx, solid, trainer=trainer)
        torch.cuda.synchronize()
        t_a = time.perf_counter()
        rho_p, u_p = trainer.predict(d)
        torch.cuda.synchronize()
        t_inf = time.perf_counter() - t_a
        lat = ws.make_lattice(gx, solid, None)
        hit0, avg0, e0 = ws_tracked(lat, u_ref, fluid)
        lat.close()
        lat = ws.make_lattice(gx, solid, None)
        k0 = ws.start_from(lat, rho_p.cpu().numpy().reshape(shape), u_p.cpu().numpy().reshape((3,) + shape))
        hit1, avg1, e1 = ws_tracked(lat, u_ref, fluid, steps0=k0)
        lat.close()
        nref = torch.linalg.vector_norm(u_ref[:, fluid])
        pred_err = float(torch.linalg.vector_norm((u_p.reshape((3,) + shape) - u_ref)[:, fluid]) / nref)
        sps0, sps1 = secs0 / max(n0, 1), (secs1 - t_inf) / max(n1, 1)
        row = dict(seed=s, gx=gx, solid_frac=frac, ref_steps=n_ref, ref_resid=r_ref, infer_secs=t_inf,
                   pred_err=pred_err, steps_rest=n0, steps_warm=n1, secs_rest=secs0, secs_warm=secs1,
                   err_end_rest=e0[0], err_end_warm=e1[0], avgerr_end_rest=e0[1], avgerr_end_warm=e1[1])
        for tg in TARGETS:
            k = "%.0e" % tg
            for key, h0, h1 in (("", hit0, hit1), ("avg_", avg0, avg1)):
                row["steps_rest_" + key + k] = h0.get(tg)
                row["steps_warm_" + key + k] = h1.get(tg)
                row["secs_rest_" + key + k] = None if tg not in h0 else h0[tg] * sps0
                row["secs_warm_" + key + k] = None if tg not in h1 else t_inf + h1[tg] * sps1
        rows.append(row)
        log("seed %d: pred err %.3f; residual 1e-6: rest %d steps %.3f s, warm %d steps %.3f s; to error 1e-3: "
            "rest %s warm %s steps (two-step average: rest %s warm %s); inference %.1f ms"
            % (s, pred_err, n0, secs0, n1, secs1, hit0.get(1e-3), hit1.get(1e-3), avg0.get(1e-3), avg1.get(1e-3),
               1e3 * t_inf))
    return rows


def ws_summarize(rows):
    import numpy as np

    def q(key):
        v = np.array([r[key] for r in rows if r[key] is not None], dtype=float)
        if v.size == 0:
            return None
        return dict(median=float(np.median(v)), q25=float(np.percentile(v, 25)),
                    q75=float(np.percentile(v, 75)), n=int(v.size))

    def speedup(kr, kw):
        v = [r[kr] / r[kw] for r in rows if r[kr] is not None and r[kw] is not None]
        return float(np.median(v)) if v else None

    def wins(kr, kw):
        return sum(1 for r in rows if r[kw] is not None and (r[kr] is None or r[kw] < r[kr]))
    out = dict(n=len(rows), pred_err=q("pred_err"), ref_steps=q("ref_steps"), infer_secs=q("infer_secs"),
               steps_rest=q("steps_rest"), steps_warm=q("steps_warm"), secs_rest=q("secs_rest"),
               secs_warm=q("secs_warm"), speedup_residual=speedup("secs_rest", "secs_warm"),
               warm_faster_residual=wins("secs_rest", "secs_warm"))
    for tg in TARGETS:
        k = "%.0e" % tg
        for key in ("", "avg_"):
            out["steps_rest_" + key + k] = q("steps_rest_" + key + k)
            out["steps_warm_" + key + k] = q("steps_warm_" + key + k)
            out["speedup_" + key + k] = speedup("secs_rest_" + key + k, "secs_warm_" + key + k)
            out["warm_faster_" + key + k] = wins("secs_rest_" + key + k, "secs_warm_" + key + k)
    out["err_end_warm"] = q("err_end_warm")
    out["avgerr_end_warm"] = q("avgerr_end_warm")
    out["err_end_rest"] = q("err_end_rest")
    return out


def warmstart_study(train=512, test=64, epochs=30, batch=4, lr=1e-3, concurrent=8, out=None):
    from paper_1007_1388_amd import warmstart as ws
    log = lambda m: print(m, flush=True)
    t0 = time.perf_counter()
    data = ws.generate(list(range(train)), concurrent=concurrent, log=log)
    t_gen = time.perf_counter() - t0
    log("generation %.1f s" % t_gen)
    tr = ws.Trainer(batch=batch)
    tr.prepare(data)
    info = tr.train(data, epochs=epochs, lr=lr, log=log)
    for d in data:
        d.clear()
    rows = ws_evaluate(tr, list(range(10000, 10000 + test)), log=log)
    rep = dict(study="warmstart", train_samples=train, test_samples=test, epochs=epochs, batch=batch,
               generation_seconds=t_gen, training=info, scale=tr.scale, summary=ws_summarize(rows),
               forward_gflop_per_sample=tr.net.flops_forward() / batch / 1e9)
    log(json.dumps(rep["summary"]))
    if out:
        rep["rows"] = rows
        with open(out, "w") as fh:
            json.dump(rep, fh, indent=1)


# ------------------------------------------------------------ convolutions
def conv_layers(n=8, D=128, H=64, W=64, reps=20):
    """Per-layer times of the three convolution kernels at the given shape
    (HIP events on the current stream): TFLOP/s (2 * voxels * taps * Cin *
    Cout per kernel).  As training runs them: activations of a random input,
    random output gradients, input gradients masked by ReLU' (stride 2: added to
    what is there), weight gradients with the bias and their ordered sums."""
    import torch
    from paper_1007_1388_amd import surrogate as S
    net = S.UNet(n, D, H, W, seed=1)
    g = torch.Generator(device="cuda").manual_seed(1)

    def fill(act, scale):
        v = scale * torch.randn(act.buf.shape, generator=g, device="cuda")
        act.buf.copy_(v.bfloat16().view(torch.int16))
    fill(net.x, 1.0)
    net.forward()
    torch.cuda.synchronize()
    st = torch.cuda.current_stream()
    L = S.lib()
    rows = []

    def timed(fn):
        fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(st)
        for _ in range(reps):
            fn()
        e1.record(st)
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    for name, l, x, y in net.io():
        dx, dy = S.Act(x.n, x.d, x.h, x.w, x.c), S.Act(y.n, y.d, y.h, y.w, y.c)
        fill(dy, 1e-3)
        fl = l.flops(y.n * y.d * y.h * y.w)
        t_f = timed(lambda: l.forward(x, y))
        t_d = timed(lambda: S._ck(L.lbm_conv3d_bwd_data(dy.ref, l.wt.data_ptr(), dx.ref, x.ref, l.k, l.stride,
                                                          1 if l.stride == 2 else 0, None), "lbm_conv3d_bwd_data"))
        t_w = timed(lambda: l.backward(x, dy, None))
        r = dict(study="conv", layer=name, cin=l.cin, cout=l.cout, k=l.k, stride=l.stride, out=(y.d, y.h, y.w),
                 gflop=fl / 1e9, fwd_ms=t_f, bwd_data_ms=t_d, bwd_weight_ms=t_w, fwd_tflops=fl / t_f / 1e9,
                 bwd_data_tflops=fl / t_d / 1e9, bwd_weight_tflops=fl / t_w / 1e9)
        rows.append(r)
        print(json.dumps(r), flush=True)
        del dx, dy
    tot = sum(r["gflop"] for r in rows)
    for kind in ("fwd", "bwd_data", "bwd_weight"):
        t = sum(r[kind + "_ms"] for r in rows)
        print(json.dumps(dict(study="conv", total=kind, gflop=tot, ms=t, tflops=tot / t)), flush=True)


def persistent_sweep(steps=2000):
    """Graph-launched steps against the persistent multi-step sweep
    (lbm_step_persistent) on small and large domains: microseconds per step."""
    import torch
    p5 = inputs.preset("warmstart")
    cases = [("cavity32 32^3 FP64", dict(dims=(32, 32, 32), walls=(True, True, True), wall_u={"+z": (0.05, 0, 0)},
                                         tau=0.6), "f64", None, None),
             ("porous 64x64x128 FP32", dict(dims=p5["dims"], walls=p5["walls"], tau=p5["tau"], force=(1e-6, 0, 0)),
              "f32", None, inputs.porous_spheres(p5["dims"], 0.12, (3, 8), seed=1)),
             ("periodic 128^3 FP32", dict(dims=(128, 128, 128), walls=(False, False, True), tau=0.8,
                                          force=(1e-6, 0, 0)), "f32", None, None),
             ("periodic 128^3 FP32, 8 Blocks", dict(dims=(128, 128, 128), walls=(False, False, True), tau=0.8,
                                                   force=(1e-6, 0, 0)), "f32",
              inputs.uniform_blocks((128, 128, 128), (2, 2, 2)), None),
             ("poiseuille 256^3 FP32", dict(dims=(256, 256, 256), walls=(False, False, True), tau=0.8,
                                           force=(1e-6, 0, 0)), "f32", None, None)]
    for label, kw, prec, blocks, solid in cases:
        for mode, arg in (("graph", 10), ("graph", 50), ("persistent", 100), ("persistent", 1000)):
            lat = lbm.Lattice(kw["dims"], blocks=blocks, walls=kw["walls"], wall_u=kw.get("wall_u"), tau=kw["tau"],
                              force=kw.get("force", (0, 0, 0)), precision=prec)
            if solid is not None:
                lat.set_geometry(solid)
            if mode == "graph":
                lat.set_schedule(graph_steps=arg)
                run = lambda n: lat.step(n)
            else:
                run = lambda n: lat.step_persistent(n, steps_per_launch=arg)
            run(100)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            run(steps)
            torch.cuda.synchronize()
            us = (time.perf_counter() - t0) * 1e6 / steps
            nf = lat.info()["n_fluid"]
            lat.sums()
            lat.close()
            print(json.dumps(dict(study="persistent", case=label, mode=mode,
                                  **({"graph_steps": arg} if mode == "graph" else {"steps_per_launch": arg}),
                                  us_per_step=round(us, 2), mlups=round(nf / us, 1))), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("study", choices=["size", "blocks", "open", "pad", "hbm", "hetero", "precision", "warmstart",
                                      "conv", "persistent"])
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--sizes", default="64-512:32")
    ap.add_argument("--n", type=int, default=384, help="precision: cavity edge")
    ap.add_argument("--train", type=int, default=512, help="warmstart: training samples")
    ap.add_argument("--test", type=int, default=64, help="warmstart: held-out seeds")
    ap.add_argument("--epochs", type=int, default=30, help="warmstart: training epochs")
    ap.add_argument("--out", default=None, help="warmstart: JSON report with every row")
    args = ap.parse_args()
    import torch
    torch.cuda.init()
    if args.study == "size":
        lo, rest = args.sizes.split("-")
        hi, st = rest.split(":")
        size_sweep(args.steps, range(int(lo), int(hi) + 1, int(st)))
    elif args.study == "open":
        open_sweep(args.steps)
    elif args.study == "pad":
        pad_sweep(args.steps)
    elif args.study == "hbm":
        hbm_sweep()
    elif args.study == "hetero":
        hetero_sweep(args.steps)
    elif args.study == "precision":
        precision_study(n=args.n)
    elif args.study == "warmstart":
        warmstart_study(train=args.train, test=args.test, epochs=args.epochs, out=args.out)
    elif args.study == "conv":
        conv_layers()
    elif args.study == "persistent":
        persistent_sweep()
    else:
        block_sweep(args.steps)


if __name__ == "__main__":
    main()
