// libsv host: programs on small tiles (sv_tile.hip), for states that the large
// tiles cannot spread over the chip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "sv_host.h"

// Tile bits of a state, 0: the large tiles.  A state of up to 13 qubits is one
// tile, and its whole program one launch.  Above that the tiles are the
// smallest that leave two tile groups (T + T - 3 qubits with runs of eight
// amplitudes), i.e. one pass per layer, which gives 16 to 512 workgroups where
// the large tiles give 2 to 256.
int tile_bits(int n, sv_dtype dt) {
    const int t = knob_for("tile", (int)dt, n);
    if (t == 0) return 0;
    if (t > 0) return (t >= 10 && t <= 13 && n <= 2 * t - 3) ? t : 0;
    if (n <= 13) return std::max(n, 10);
    if (n > 21) return 0;
    return std::max(10, (n + 4) / 2);
}

// Energy table E(z) of an instance, followed by kEtabTail doubles of scratch (built once, on the
// caller's stream, which is synchronised so that later launches on any stream may read it; wait =
// false: the caller synchronises it).
constexpr size_t kEtabTail = 4;
static int get_etab(sv_ising_s* H, hipStream_t stream, const double** out, bool lookup_only, bool wait = true) {
    std::lock_guard<std::mutex> g(H->mu);
    if (!H->d_etab) {
        if (lookup_only)
            return fail(SV_ERR_UNSUPPORTED, "the instance has no energy table yet (run sv_qaoa_energy once with a state "
                                            "of the same n and dtype to build it)");
        double* d = nullptr;
        HIPCHECK(hipMalloc(&d, (sizeof(double) << H->n) + kEtabTail * sizeof(double)));
        int e = launch_energy_table(ising_dev(H), d, stream);
        if (e == 0 && wait) e = (int)hipStreamSynchronize(stream);
        if (e != 0) {
            (void)hipFree(d);
            return fail(SV_ERR_HIP, "energy table build failed: %s", hipGetErrorString((hipError_t)e));
        }
        H->d_etab = d;
    }
    *out = H->d_etab;
    return SV_OK;
}

// Records a small-tile pass as a run of it would (tile_seen) and builds the energy table it reads.
int prepare_tile_pass(sv_ising_s* H, hipStream_t stream, int dt, int T, int group, bool point) {
    const double* E = nullptr;
    int rc = get_etab(H, stream, &E, false);
    if (rc) return rc;
    std::lock_guard<std::mutex> g(H->mu);
    H->tile_seen.insert(std::make_tuple(dt, T, group, point));
    if (point) H->tile_seen.insert(std::make_tuple(dt, T, group, false));
    return SV_OK;
}

// Ground states of a state of up to 14 qubits, from the energy table that its evaluations read (the
// enumeration over tiles or an independent set would build tables of its own beside it: a new
// instance and its ground states, n = 10, real couplings 305 -> 154 us, 3-regular 301 -> 154 us).
// Complex64 evaluations that may not build tables (tile_seen) follow this call alone.
int run_ground_table(sv_ising_s* H, hipStream_t stream, int T) {
    const double* E = nullptr;
    int rc = get_etab(H, stream, &E, false, false);
    if (rc) return rc;
    double* const d_out = H->d_etab + ((size_t)1 << H->n);
    double res[3] = {0.0, 0.0, 0.0};
    int e = launch_ground_table(E, H->n, ground_tol(H), d_out, stream);
    if (!e) e = (int)hipMemcpyAsync(res, d_out, sizeof(res), hipMemcpyDeviceToHost, stream);
    if (!e) e = (int)hipStreamSynchronize(stream);
    if (e) return fail(SV_ERR_HIP, "ground enumeration failed: %s", hipGetErrorString((hipError_t)e));
    std::lock_guard<std::mutex> g(H->mu);
    H->emin = res[0];
    H->deg = (uint64_t)res[1];
    H->argmin = (uint64_t)res[2];
    H->has_ground = true;
    for (int grp = 0; grp < 2; grp++)
        for (bool point : {false, true}) H->tile_seen.insert(std::make_tuple((int)SV_C64, T, grp, point));
    return SV_OK;
}

// 4 J over the pairs of register bits set in r, for the layout that starts at tile bit b.
static void register_couplings(const Geometry& geo, const sv_ising_s* H, int b, double* Q) {
    int slot[64];
    for (int& x : slot) x = -1;
    for (int k = 0; k < kTileR; k++) {
        const int l = b + k;
        if (l < geo.n) slot[l < geo.c ? l : geo.lo + (l - geo.c)] = k;
    }
    for (int e = 0; e < H->m; e++) {
        const int ka = slot[H->ei[e]], kb = slot[H->ej[e]];
        if (ka < 0 || kb < 0) continue;
        for (int r = 0; r < (1 << kTileR); r++)
            if ((r >> ka & 1) && (r >> kb & 1)) Q[r] += 4.0 * H->J[e];
    }
}

// Phase angles within the range of the in-place phase factors (an exponent is at most
// 4 |gamma| (sum|h| + sum|J|)).
bool small_angles(const sv_ising_s* H, int p, const double* gamma) {
    double g = 0.0;
    for (int k = 0; k < p; k++) g = std::max(g, std::fabs(gamma[k]));
    return 4.0 * g * H->scale <= kTileMaxAngle;
}
static bool small_angles(const sv_ising_s* H, const Program& prog) {
    for (const Pass& p : prog.passes)
        for (const auto& ph : p.phase)
            if (!small_angles(H, 1, &ph.second)) return false;
    return true;
}

// Calls that may not build tables evaluate energies on the small tiles whatever their angles: a
// program of the same state that ran on the large tiles instead (angles, or more results than a
// small-tile program can have) prepares them as one on the small tiles would.
int prepare_tile_passes(sv_state_s* s, sv_ising_s* H, const Plan& plan) {
    const int tb = plan.tile ? 0 : tile_bits(s->n, s->dt);
    for (int grp = 0; tb > 0 && grp < 2; grp++) {
        int rc = prepare_tile_pass(H, s->stream, (int)s->dt, tb, grp, true);
        if (rc) return rc;
    }
    return SV_OK;
}

// One launch: a list of ops on the tiles of one group.
struct TileLaunch {
    int group = 0, nv = 1, load = 1, store = 1;
    std::vector<TileOp> ops;
    std::vector<int> layer;  // per op: general layer index or -1
    bool real = false;       // its ops are general layers with real matrices
};

int run_tile_program(sv_state_s* s, sv_state_s* lam, sv_ising_s* H, Program& prog, const Plan& plan, bool need_ground,
                     const FixedScratch* fx, const void* first_src, bool dual) {
    if (s->failed) return fail(SV_ERR_HIP, "state is in a failed state after an earlier HIP error");
    if (!fx) {
        int rc = drop_results(s);
        if (rc) return rc;
    }
    const std::vector<Geometry>& groups = plan.by_nv[1];
    const int T = groups[0].T;
    const uint64_t ntiles = groups[0].ntiles;
    const bool single = groups.size() == 1;  // one tile holds the state: results need no second stage
    double emin = 0.0, etol = 0.0;
    if (need_ground && H) {
        if (fx) {
            std::lock_guard<std::mutex> g(H->mu);
            if (!H->has_ground)
                return fail(SV_ERR_UNSUPPORTED, "the instance has no ground-state cache yet (call sv_ground once)");
        } else {
            int rc = run_ground(H, s->stream);
            if (rc) return rc;
        }
        emin = H->emin;
        etol = ground_tol(H);
    }
    if (fx) {
        // the limits of the call (they also bound what the large tiles keep in the fixed region)
        size_t tab = 0;
        std::lock_guard<std::mutex> g(H->mu);
        for (const Pass& p : prog.passes) {
            tab += p.phase.size() * (32 + (size_t)(H->lut_half >= 0 ? 2 * H->lut_half + 1 : 0));
            bool point = false;
            for (const Op& op : p.ops) point = point || op.kind == OP_POINT;
            if (!H->tile_seen.count(std::make_tuple((int)s->dt, T, p.group, point)))
                return fail(SV_ERR_UNSUPPORTED, "the instance has no device tables for this n, dtype and plan yet (run "
                                                "sv_qaoa_energy once with a state of the same n and dtype to build them)");
        }
        if (tab > fx->tab_entries)
            return fail(SV_ERR_UNSUPPORTED, "phase tables need %zu entries, the fixed scratch holds %zu", tab,
                        fx->tab_entries);
    }

    // launches and result columns
    std::vector<TileLaunch> launches;
    std::vector<std::vector<uint32_t>> segs(std::max(prog.nres, 0));  // per result: its columns (GatherArgs::seg)
    int ncol = 0, nblk = 0, feat = 0;
    bool uses_e = false;
    for (const Pass& p : prog.passes) {
        // columns of the pass's slots
        std::vector<int> col(p.slot_dst.size());
        for (size_t q = 0; q < col.size(); q++) {
            col[q] = single ? p.slot_dst[q] : ncol++;
            if (!single) segs[p.slot_dst[q]].push_back((uint32_t)col[q] | 255u << 24);
        }
        int spin = -1;
        if (p.spin_res >= 0) {
            spin = single ? p.spin_res : ncol;
            if (!single) {
                spin_segments(groups[p.group], s->n, ncol, ncol + T, &segs[p.spin_res]);
                ncol += T + 1;
            }
        }
        int nops = 0;
        for (const Op& op : p.ops) nops += op.kind != 0;
        const bool join = single && !launches.empty() && (int)launches.back().ops.size() + nops <= kMaxTileOps &&
                          launches.back().nv == p.nv && !p.init;
        if (!join) {
            launches.emplace_back();
            launches.back().group = p.group;
            launches.back().nv = p.nv;
            launches.back().load = p.load;
        }
        TileLaunch& L = launches.back();
        L.store = p.store;
        bool point = false;
        for (const Op& op : p.ops) {
            if (op.kind == 0) continue;
            TileOp o{};
            o.w0 = (uint32_t)op.kind | (uint32_t)op.flags << 8;
            o.parts = ((uint32_t)(op.slot >= 0 ? col[op.slot] : 0) & 0xffffu) |
                      (uint32_t)(op.slot2 >= 0 ? col[op.slot2] : 0) << 16;
            o.aux = -1;
            o.a = op.a;
            o.b = op.b;
            int layer = -1;
            if (op.kind == OP_MIX && (op.flags & MIX_GEN)) {
                layer = op.qidx;
                o.aux = nblk++;
                feat |= 2;
            }
            if (op.kind == OP_MIX && (op.flags & MIX_GBETA)) feat |= 1;
            if (op.kind == OP_POINT) {
                point = true;
                uses_e = uses_e || H;
                if (op.flags & PT_SPINZ) {
                    o.aux = spin;
                    feat |= 2;
                }
                if (op.flags & (PT_ZETA | PT_EFORM | PT_LAM_INIT | PT_GGAMMA)) feat |= 1;
                if (op.flags & PT_E2) return fail(SV_ERR_UNSUPPORTED, "internal: point op without a small-tile form");
            }
            L.ops.push_back(o);
            L.layer.push_back(layer);
        }
        if (H && !fx) {
            std::lock_guard<std::mutex> g(H->mu);
            H->tile_seen.insert(std::make_tuple((int)s->dt, T, p.group, point));
            if (point) H->tile_seen.insert(std::make_tuple((int)s->dt, T, p.group, false));
        }
        if (L.nv == 2 && !lam) return fail(SV_ERR_ARG, "internal: two-vector pass without lam");
    }
    if (ncol > kMaxTileColumns || prog.nres * (dual ? 2 : 1) > kMaxTileColumns || feat == 3)
        return fail(SV_ERR_UNSUPPORTED, "internal: program does not fit the small tiles");
    if (H && !small_angles(H, prog)) {
        if (feat != 0) return fail(SV_ERR_UNSUPPORTED, "internal: phase angles beyond the small tiles");
        feat = 3;
    }
    if (dual && (!single || launches.size() != 1))
        return fail(SV_ERR_UNSUPPORTED, "internal: a paired program needs one launch");

    // workspaces
    const double* E = nullptr;
    if (uses_e) {
        int rc = get_etab(H, s->stream, &E, fx != nullptr);
        if (rc) return rc;
    }
    const size_t part_need = single ? 1 : (size_t)ncol * ntiles;
    const int nres = prog.nres * (dual ? 2 : 1);
    double *part = nullptr, *out = nullptr;
    if (fx) {
        if (part_need > fx->part_doubles)
            return fail(SV_ERR_UNSUPPORTED, "reduction partials need %zu doubles, the fixed scratch holds %zu", part_need,
                        fx->part_doubles);
        if (nblk > 0) return fail(SV_ERR_UNSUPPORTED, "general layers need allocated scratch");
        part = fx->part;
        out = fx->out;
    } else {
        int rc = ensure_work(s, part_need, std::max(nres, 1));
        if (rc) return rc;
        part = s->w.d_part;
        // the last stage writes the results to the pinned host buffer, from which fetch_results reads
        // them as they arrive (gather_results) or after the stream (one tile)
        out = s->w.h_res;
        s->w.res_on_host = true;
    }
    if (nblk > 0) {
        if (!prog.layers || prog.nq != s->n) return fail(SV_ERR_ARG, "internal: general layers without matrices");
        double* h = nullptr;
        int rc = stage_matrices(s, (size_t)nblk, &h);
        if (rc) return rc;
        for (TileLaunch& L : launches) {
            L.real = L.nv == 1 && !L.ops.empty();
            for (size_t i = 0; i < L.ops.size(); i++) {
                if (L.layer[i] < 0) {
                    L.real = false;
                    continue;
                }
                const Geometry& geo = groups[L.group];
                double* blk = h + (size_t)L.ops[i].aux * kGenBlock;
                for (int l = 0; l < kGenBlock / 8; l++) {
                    const int q = l < T && l < s->n ? (l < geo.c ? l : geo.lo + (l - geo.c)) : -1;
                    const double id[8] = {1, 0, 0, 0, 0, 0, 1, 0};
                    memcpy(blk + 8 * l, q < 0 ? id : prog.layers + ((size_t)L.layer[i] * s->n + q) * 8, 8 * sizeof(double));
                    for (int x = 1; x < 8; x += 2) L.real = L.real && blk[8 * l + x] == 0.0;
                }
            }
        }
        rc = send_matrices(s, (size_t)nblk);
        if (rc) return rc;
    }

    for (size_t li = 0; li < launches.size(); li++) {
        TileLaunch& L = launches[li];
        const Geometry& geo = groups[L.group];
        TileArgs a;
        memset(&a, 0, sizeof(a));
        a.psi = s->ptr;
        a.lam = lam ? lam->ptr : nullptr;
        a.src = li == 0 ? first_src : nullptr;
        a.part = single ? out : part;
        a.gmat = s->w.d_gmat;
        a.ntiles = ntiles;
        a.n = s->n;
        a.c = geo.c;
        a.lo = geo.lo;
        a.g = geo.g;
        a.phantom = geo.phantom;
        a.nlayouts = (int)geo.blocks.size();
        for (int j = 0; j < a.nlayouts; j++) {
            a.lbpack |= (uint32_t)(geo.blocks[j][0] | geo.pairs[j] << 4) << (8 * j);
            a.act |= (geo.act_fwd[j] | geo.dpp[j]) << (8 * j);
        }
        a.load = L.load;
        a.store = dual ? 0 : L.store;
        a.nops = (int)L.ops.size();
        a.spin_cols = single ? s->n : T + 1;
        a.dual = dual ? 1 : 0;
        a.dual_cols = prog.nres;
        a.resident = single ? 1 : 0;
        a.feat = L.nv == 2 ? 1 : L.real ? 4 : feat;
        if (H && H->qden > 0 && H->scale * H->qden < kTileLut) {
            // every energy is sum |h| + sum |J| less an even multiple of 1 / q
            a.lut_n = (int)(H->scale * H->qden) + 1;
            a.lut_step = 1.0 / H->qden;
        }
        a.emin = emin;
        a.etol = etol;
        a.amp0 = std::pow(2.0, -0.5 * s->n);
        int cur = 0;
        for (int i = 0; i < a.nops; i++) {
            a.ops[i] = L.ops[i];
            if ((L.ops[i].w0 & 255u) == (uint32_t)OP_MIX) {
                if (a.nlayouts > 1) cur ^= 1;
            } else if (H) {
                a.need_e |= cur ? 2 : 1;
            }
        }
        a.E = E;
        if (H && a.need_e) {
            register_couplings(geo, H, geo.blocks[0][0], a.Q[0]);
            register_couplings(geo, H, geo.blocks[a.nlayouts - 1][0], a.Q[1]);
        }
        hipEvent_t ev0;
        const bool prof = !fx && prof_begin(s->stream, &ev0);
        const int e = take_injected_failure() ? (int)hipErrorLaunchFailure
                                              : launch_tile((int)s->dt, L.nv, T, a, s->stream);
        if (prof) {
            const int nrd = (a.load & 4) ? 0 : __builtin_popcount(a.load & 3);
            const int nwr = __builtin_popcount(a.store & 3);
            prof_end(s->stream, ev0, std::string("pass_") + (s->dt == SV_C128 ? "c128" : "c64") + "_nv" +
                                         std::to_string(L.nv) + "/T" + std::to_string(T) + "c" + std::to_string(geo.c) +
                                         (geo.g > 0 ? "o" + std::to_string(geo.lo) : "") + "L" +
                                         std::to_string(a.nlayouts) + ((a.load & 4) ? "w" : ""),
                     (double)(nrd + nwr) * (double)s->bytes);
        }
        if (e != 0) {
            s->failed = true;
            return fail(SV_ERR_HIP, "pass launch failed: %s", hipGetErrorString((hipError_t)e));
        }
    }
    if (single || prog.nres == 0) return SV_OK;
    return gather_results(s, part, ntiles, out, segs);
}

void spin_segments(const Geometry& geo, int n, int col, int norm, std::vector<uint32_t>* segs) {
    for (int i = 0; i < n; i++) {
        const bool in = i < geo.c || (i >= geo.lo && i < geo.lo + geo.g);
        const int l = i < geo.c ? i : geo.c + (i - geo.lo);        // tile bit
        const int w = i < geo.lo ? i - geo.c : i - geo.g - geo.c;  // bit of the tile index
        segs[i].push_back(in ? (uint32_t)(col + l) | 255u << 24 : (uint32_t)norm | (uint32_t)w << 24);
    }
}

int gather_results(sv_state_s* s, const double* part, uint64_t ntiles, double* out,
                   const std::vector<std::vector<uint32_t>>& segs) {
    if (out == s->w.h_res) {
        for (size_t i = 0; i < segs.size(); i++) memcpy(out + i, &kAwaited, sizeof(double));
        s->w.awaited = (int)segs.size();
    }
    for (size_t r0 = 0; r0 < segs.size();) {
        GatherArgs ga;
        ga.part = part;
        ga.out = out + r0;
        ga.ntiles = (uint32_t)ntiles;
        int n = 0, k = 0;
        while (r0 + n < segs.size() && n < 256 && k + (int)segs[r0 + n].size() <= 768) {
            ga.first[n] = (uint16_t)k;
            for (uint32_t sg : segs[r0 + n]) ga.seg[k++] = sg;
            n++;
        }
        if (n == 0) return fail(SV_ERR_UNSUPPORTED, "internal: a result with too many columns");
        ga.first[n] = (uint16_t)k;
        const int e = launch_gather(ga, n, s->stream);
        if (e != 0) {
            s->failed = true;
            return fail(SV_ERR_HIP, "reduce launch failed: %s", hipGetErrorString((hipError_t)e));
        }
        r0 += n;
    }
    return SV_OK;
}
