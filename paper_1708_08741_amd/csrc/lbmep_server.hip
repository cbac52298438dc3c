// lbmep_server.hip -- request server: continuous batching of independent
// lattice Boltzmann simulations on one GPU (the C ABI lbmep_server_* of
// include/lbmep.h).
//
// Requests are queued on submit (all inputs copied).  A request is admitted
// (FIFO) when a slot is free and its device footprint fits the budget; its
// lattice is then built inside one pre-allocated device arena, so admission
// and retirement never call hipMalloc / hipFree (whose implicit device
// synchronisation would drain the pipeline of the other simulations); the
// fields of finished requests lie in pinned slabs that are kept.  Set-up
// runs on its own stream while the resident simulations keep stepping.
//
// Resident simulations advance together in chunks of steps.  Every step of a
// chunk is two packed launches per (precision, force mode): the sweep with the
// mapping of the next level, and the bounce-back / exchange with its
// classification (three with many particles), each over every resident
// lattice, a workgroup finding its lattice through a block table in the kernel
// arguments.  A simulation whose last step is in a chunk has its results
// (force and torque of the last step, FP64 mass / momentum of the final
// state, optionally the fields) computed right after that chunk on the same
// stream; when the host sees the completion event it copies them out and
// releases the lattice's memory to the arena.
//
// The arithmetic is that of the single-lattice path (the same device code):
// a simulation's fields, forces and torques are bitwise the same alone and
// in any mix (the per-particle sums are fixed-order wavefront and workgroup
// sums, no atomics).
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <deque>
#include <map>
#include <memory>
#include <thread>
#include <unordered_map>

#include "first_fit.h"
#include "lattice.h"

using namespace lbmep;
using namespace lbmep::rt;

namespace {

// the one device allocation that the lattices live in
class Arena final : public DevHeap {
  public:
    static constexpr size_t kAlign = FirstFit::kAlign;

    ~Arena() override {
        if (base_) hipFree(base_);
    }
    hipError_t init(size_t bytes) {
        fit_ = FirstFit(bytes);
        const hipError_t e = hipMalloc(&base_, fit_.size());
        if (e != hipSuccess) base_ = nullptr;
        return e;
    }
    void *alloc(size_t bytes) override {
        const size_t off = fit_.alloc(bytes);
        return off == FirstFit::kNone ? nullptr : base_ + off;
    }
    void release(void *p) override {
        if (p) fit_.release((size_t)(static_cast<char *>(p) - base_));
    }
    size_t used() const { return fit_.used(); }
    size_t size() const { return fit_.size(); }

  private:
    char *base_ = nullptr;
    FirstFit fit_;
};

// Pinned host memory for the results of one server.  A copy from the device
// into pinned memory runs beside the host and the stepping at the link's rate
// (32 MB: 0.6 ms; into fresh pageable memory 8 ms, with the host waiting).
// The memory is pinned in slabs of kSlab (or one result's size), each when the
// results no longer fit in those there are, all together below `limit`; a
// result that finds no room goes to pageable memory.  Pinning takes the
// stepping thread's time, and the first read of a new slab too, so the first
// results of a server pay for the slabs and later ones of whatever size use
// them again.  A slab goes back with the server and not before: to free it
// could wait for the device, in the middle of the stepping.  Eight FP32 requests
// of 72^3 to 96^3 cells, waiting for them and reading their 8 to 28 MB each: into
// pageable memory 51 + 11 ms; here the first batch of a process 37 + 28, of a
// further server 13 + 19, every later one 13 + 6.  160 results of 0.4 to 12 MB,
// 24 of them held, near the limit: 213 ms, and 257 with a block per result that
// is freed to make room.
class PinnedBlocks {
  public:
    static constexpr size_t kSlab = size_t(32) << 20;

    ~PinnedBlocks() {
        for (auto &s : slabs_) hipHostFree(s.first);
    }
    void set_limit(size_t bytes) { limit_ = bytes; }
    double *take(size_t bytes) {
        for (auto &s : slabs_) {
            const size_t off = s.second.alloc(bytes);
            if (off != FirstFit::kNone) return reinterpret_cast<double *>(s.first + off);
        }
        const size_t need = round_up(bytes, FirstFit::kAlign);
        const size_t room = limit_ > held_ ? limit_ - held_ : 0;
        if (need > room) return nullptr;
        const size_t slab = std::max(need, std::min(kSlab, room / FirstFit::kAlign * FirstFit::kAlign));
        void *p = nullptr;
        if (hipHostMalloc(&p, slab, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        FirstFit &f = slabs_.emplace(static_cast<char *>(p), FirstFit(slab)).first->second;
        held_ += slab;
        return reinterpret_cast<double *>(static_cast<char *>(p) + f.alloc(bytes));
    }
    void give(double *p) {
        if (!p) return;
        auto it = std::prev(slabs_.upper_bound(reinterpret_cast<char *>(p)));
        it->second.release((size_t)(reinterpret_cast<char *>(p) - it->first));
    }

  private:
    size_t limit_ = 0, held_ = 0;
    std::map<char *, FirstFit> slabs_;
};

struct Request {
    uint64_t id = 0;
    lbmep_config cfg{};
    std::vector<uint8_t> flags;
    int32_t n = 0, steps = 0;
    std::vector<double> X, R, U, W;
    std::vector<char> rho_e;
    int32_t rho_dtype = 0;
    bool charge = false, keep_fields = false;
    double E[3] = {0, 0, 0};
    size_t footprint = 0;
    bool tight = false;  // admitted in the tight form
    double t_submit = 0, t_admit = 0, t_done = 0;
    // results
    bool done = false;
    int status = LBMEP_OK;
    std::string error;
    std::vector<double> F, M, rho, u;
    double *fields = nullptr;  // rho, u in a pinned block (instead of the vectors)
    double inv[4] = {0, 0, 0, 0};
};

struct Slot {
    Request *req = nullptr;
    lbmep_lattice *L = nullptr;
    LatticeDev *d = nullptr;   // device descriptor (in the arena)
    int32_t to_enqueue = 0;    // steps not yet enqueued
    bool retiring = false;     // result read-out enqueued, waiting for its event
    hipEvent_t ev = nullptr;
    double *fields = nullptr;  // rho, u of the final state (arena), keep_fields only
};

double now_s(std::chrono::steady_clock::time_point t0) {
    return std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
}

bool small_offsets(const lbmep_config &c) {
    const size_t N = (size_t)c.nx * c.ny * c.nz;
    const size_t Ns = population_stride(N, c.precision);
    return 2 * Ns * storage_bytes(c.precision) < (size_t(1) << 32) && 4 * Ns < (size_t(1) << 32);
}

}  // namespace

struct lbmep_server {
    lbmep_server_config cfg{};
    std::chrono::steady_clock::time_point t0;
    Arena arena;
    PinnedBlocks pinned;
    hipStream_t main = nullptr, setup = nullptr, copy = nullptr;
    std::deque<std::unique_ptr<Request>> queue;
    std::unordered_map<uint64_t, std::unique_ptr<Request>> finished;
    std::deque<uint64_t> unreported;  // finished ids not yet returned by poll
    std::vector<Slot> slots;
    std::deque<hipEvent_t> chunk_ev;  // completion events of enqueued chunks
    std::deque<double> chunk_work;    // their cell updates
    std::vector<hipEvent_t> ev_pool;
    uint64_t next_id = 1;
    size_t reserved = 0;  // footprints of the resident requests
    lbmep_server_stats st{};
};

namespace {

// copy of a result into the caller's memory, which is mostly touched here for
// the first time: a large one by four threads (eight results of 30 MB on
// average: one thread 13.5 ms, four 7.6 ms)
void copy_out(void *dst, const void *src, size_t bytes) {
    constexpr size_t kParts = 4, kLarge = size_t(4) << 20;
    const size_t part = bytes < kLarge ? bytes : round_up(bytes / kParts + 1, 4096);
    std::vector<std::thread> t;
    size_t done = 0;
    try {
        t.reserve(kParts);
        for (; done + part < bytes; done += part)
            t.emplace_back(std::memcpy, static_cast<char *>(dst) + done,
                           static_cast<const char *>(src) + done, part);
    } catch (...) {  // no thread to be had: the rest is copied here
    }
    std::memcpy(static_cast<char *>(dst) + done, static_cast<const char *>(src) + done, bytes - done);
    for (std::thread &k : t) k.join();
}

hipEvent_t get_event(lbmep_server *S) {
    if (!S->ev_pool.empty()) {
        hipEvent_t e = S->ev_pool.back();
        S->ev_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return nullptr;
    return e;
}

size_t request_footprint(const lbmep_config &c, int32_t n, double r_max, bool charge, bool flags,
                         bool keep_fields, bool tight) {
    const size_t N = (size_t)c.nx * c.ny * c.nz;
    size_t b = lattice_bytes(&c, n, r_max, charge ? kForceCharge : kForceNone, tight);
    b += 32 * Arena::kAlign;                 // alignment of the lattice's arrays
    if (!tight) b += round_up(sizeof(LatticeDev), Arena::kAlign);
    // staging of the inputs during set-up
    size_t stage = 0;
    if (flags) stage = std::max(stage, N);
    if (charge) stage = std::max(stage, N * sizeof(double));
    b += round_up(stage, Arena::kAlign);
    if (keep_fields) b += round_up(4 * N * sizeof(double), Arena::kAlign);
    return b;
}

void fail_request(Request *r, int code, const std::string &msg) {
    r->status = code;
    r->error = msg;
}

// workgroups of the packed sweep that map the next level of a lattice
uint32_t map_blocks(const lbmep_lattice *L) {
    const uint32_t per = kPackBlockX / kMapThreads;
    return L->np > 0 && L->cfg.move_particles ? ((uint32_t)L->np + per - 1u) / per : 0u;
}

// build the lattice of a request on the set-up stream, take its first step
// there (it starts from a post-stream state), and write its descriptor
int admit(lbmep_server *S, Slot &slot, Request *r) {
    lbmep_config c = r->cfg;
    c.device = S->cfg.device;
    c.stream = S->setup;
    lbmep_lattice *L = nullptr;
    int rc = create_lattice(&c, &S->arena, &L);
    if (rc) return rc;
    if (r->tight) make_tight(L);
    auto undo = [&](int code) {
        destroy_lattice(L, true);
        return code;
    };
    if (!r->flags.empty()) {
        rc = lbmep_set_flags(L, r->flags.data(), 0);
        if (rc) return undo(rc);
    }
    if (r->charge) {
        rc = lbmep_set_charge_force(L, r->rho_e.data(), r->rho_dtype, r->E, 0);
        if (rc) return undo(rc);
    }
    // (a new lattice rests in equilibrium at density 1)
    rc = lbmep_set_particles(L, r->n, r->X.data(), r->R.data(), r->U.data(), r->W.data());
    if (rc) return undo(rc);
    rc = lbmep_step(L, 1);
    if (rc) return undo(rc);
    // device descriptor for the packed launches (a lattice in the tight form
    // is stepped by launches of its own)
    LatticeDev h{};
    h.split = L->overlap && L->np > 0;
    for (int cur = 0; cur < 2; ++cur)
        for (int co = 0; co < 3; ++co) {
            SweepArgs a = sweep_args_state(L, cur, co);
            if (h.split) {
                // the lists change places with the population grids
                const int l = L->lcur ^ L->cur ^ cur;
                a.plist = L->plist_buf[l];
                a.pcount = L->pcount_buf[l];
                h.plist[cur] = L->plist_buf[l ^ 1];
                h.pcount[cur] = L->pcount_buf[l ^ 1];
            }
            h.sweep[cur + 2 * co] = a;
        }
    h.pa = particle_args(L);
    for (int b = 0; b < 3; ++b) h.map[b] = L->map[b];
    h.map_blocks = map_blocks(L);
    h.wall_blocks = near_wall_blocks(L->g, L->has_walls, L->part_threads);
    LatticeDev *d = nullptr;
    if (!L->tight) {
        d = static_cast<LatticeDev *>(S->arena.alloc(sizeof(LatticeDev)));
        if (!d) return undo(fail(LBMEP_ENOMEM, "arena exhausted (descriptor)"));
    }
    double *fields = nullptr;
    if (r->keep_fields) {
        fields = static_cast<double *>(S->arena.alloc(4 * L->g.N * sizeof(double)));
        if (!fields) {
            S->arena.release(d);
            return undo(fail(LBMEP_ENOMEM, "arena exhausted (fields)"));
        }
    }
    hipError_t e = hipSuccess;
    if (d) e = hipMemcpyAsync(d, &h, sizeof h, hipMemcpyHostToDevice, S->setup);
    if (e == hipSuccess) e = hipStreamSynchronize(S->setup);
    if (e != hipSuccess) {
        S->arena.release(d);
        S->arena.release(fields);
        return undo(fail(LBMEP_EDEVICE, std::string("descriptor: ") + hipGetErrorString(e)));
    }
    // from now on the lattice's work is enqueued on the main stream
    L->stream = S->main;
    slot.req = r;
    slot.L = L;
    slot.d = d;
    slot.fields = fields;
    slot.to_enqueue = r->steps - 1;
    slot.retiring = false;
    r->t_admit = now_s(S->t0);
    return LBMEP_OK;
}

// enqueue the result read-out of a slot whose last step is enqueued
int enqueue_readout(lbmep_server *S, Slot &slot) {
    lbmep_lattice *L = slot.L;
    hipStream_t s = S->main;
    if (L->np > 0)
        LBMEP_HIP_TRY(launch_finalize_ft(L->np, L->FM, L->map[L->ft_buf].X,
                                         L->FM + 12 * (size_t)L->np, s));
    int rc = materialize(L);
    if (rc) return rc;
    double *dout = L->red + 5 * (size_t)L->red_blocks;
    LBMEP_HIP_TRY(launch_invariants(L->precision, L->g, L->f[L->cur], L->flag, L->red,
                                    L->red_blocks, dout, s));
    if (slot.fields) {
        const size_t N = L->g.N;
        LBMEP_HIP_TRY(launch_macro(L->precision, L->force_mode, sweep_args(L), L->pmode,
                                   slot.fields, slot.fields + N, s));
    }
    slot.ev = get_event(S);
    if (!slot.ev) return fail(LBMEP_EDEVICE, "event creation failed");
    LBMEP_HIP_TRY(hipEventRecord(slot.ev, s));
    if (slot.fields) {
        // the fields travel beside the stepping of the other simulations
        const size_t b = 4 * L->g.N * sizeof(double);
        slot.req->fields = S->pinned.take(b);
        if (slot.req->fields) {
            LBMEP_HIP_TRY(hipStreamWaitEvent(S->copy, slot.ev, 0));
            LBMEP_HIP_TRY(hipMemcpyAsync(slot.req->fields, slot.fields, b, hipMemcpyDeviceToHost,
                                         S->copy));
            LBMEP_HIP_TRY(hipEventRecord(slot.ev, S->copy));
        }
    }
    slot.retiring = true;
    return LBMEP_OK;
}

// copy the results of a completed slot to its request and free the slot
void retire(lbmep_server *S, Slot &slot) {
    lbmep_lattice *L = slot.L;
    Request *r = slot.req;
    const size_t N = L->g.N;
    bool ok = true;
    if (L->np > 0) {
        std::vector<double> h(6 * (size_t)L->np);
        ok = hipMemcpy(h.data(), L->FM + 12 * (size_t)L->np, h.size() * sizeof(double),
                       hipMemcpyDeviceToHost) == hipSuccess;
        r->F.resize(3 * (size_t)L->np);
        r->M.resize(3 * (size_t)L->np);
        for (int p = 0; p < L->np; ++p)
            for (int k = 0; k < 3; ++k) {
                r->F[3 * p + k] = h[6 * (size_t)p + k];
                r->M[3 * p + k] = h[6 * (size_t)p + 3 + k];
            }
    }
    ok = ok && hipMemcpy(r->inv, L->red + 5 * (size_t)L->red_blocks, 4 * sizeof(double),
                         hipMemcpyDeviceToHost) == hipSuccess;
    if (slot.fields && !r->fields) {
        r->rho.resize(N);
        r->u.resize(3 * N);
        ok = ok && hipMemcpy(r->rho.data(), slot.fields, N * sizeof(double),
                             hipMemcpyDeviceToHost) == hipSuccess;
        ok = ok && hipMemcpy(r->u.data(), slot.fields + N, 3 * N * sizeof(double),
                             hipMemcpyDeviceToHost) == hipSuccess;
    }
    if (!ok) fail_request(r, LBMEP_EDEVICE, "result copy failed");
    r->t_done = now_s(S->t0);
    r->done = true;
    S->arena.release(slot.fields);
    S->arena.release(slot.d);
    destroy_lattice(L, false);  // its work is complete (event)
    S->ev_pool.push_back(slot.ev);
    S->reserved -= r->footprint;
    S->st.completed += 1;
    S->finished[r->id].reset(r);
    S->unreported.push_back(r->id);
    slot = Slot{};
}

// enqueue `k` steps of every active slot as packed launches (those in the
// tight form, which only a budget without room for the other sees, one by one)
int enqueue_steps(lbmep_server *S, const std::vector<Slot *> &act, int k) {
    hipStream_t s = S->main;
    size_t bytes = 0;
    for (const Slot *sl : act) bytes += population_bytes(sl->L->g, sl->L->precision);
    for (int it = 0; it < k; ++it) {
        // sweep and exchange, one packed launch pair per (precision, force
        // mode); lattices of many particles apart, with a third launch for the
        // classification
        for (int prec = LBMEP_FP64; prec <= LBMEP_FP16DEV; ++prec)
            for (int kind = 0; kind < 2 * (kForceCharge + 1); ++kind) {
                const int fm = kind >> 1;
                const bool many = (kind & 1) != 0;
                const int nt = many ? kManyThreads : kPartThreads;
                PackTable ts{}, tn{}, tc{};
                uint32_t lds = near_lds(nt), rows = 0;
                int box = kPartThreads / 2;  // of the largest of the lattices
                ts.xcd_swizzle = 1;
                ts.cached = bytes < kInfinityCache;
                auto flush = [&]() -> int {
                    if (ts.n == 0) return LBMEP_OK;
                    LBMEP_HIP_TRY(launch_sweep_packed(prec, fm, ts, s));
                    LBMEP_HIP_TRY(launch_parts_packed(prec, tn, nt, lds, s));
                    if (tc.n) LBMEP_HIP_TRY(launch_classify_packed(tc, box, classify_lds(rows, box), s));
                    S->st.packed_launches += tc.n ? 3 : 2;
                    ts.n = tn.n = tc.n = 0;
                    ts.start[0] = tn.start[0] = tc.start[0] = 0;
                    lds = near_lds(nt);
                    rows = 0;
                    box = kPartThreads / 2;
                    return LBMEP_OK;
                };
                for (Slot *sl : act) {
                    lbmep_lattice *L = sl->L;
                    if (L->tight || L->precision != prec || L->force_mode != fm ||
                        (L->part_threads == kManyThreads) != many)
                        continue;
                    const bool moving = L->np > 0 && L->cfg.move_particles;
                    const uint32_t state = (uint32_t)(L->cur + 2 * L->cur_owner);
                    const uint32_t sb =
                        map_blocks(L) + (uint32_t)((L->g.N + kPackBlockX - 1) / kPackBlockX);
                    if (moving && many) {
                        box = std::max(box, L->box_threads);
                        rows = std::max(rows, L->box_rows);
                        tc.d[tc.n] = sl->d;
                        tc.state[tc.n] = state;
                        tc.start[tc.n + 1] = tc.start[tc.n] + (uint32_t)L->np;
                        tc.n++;
                    } else if (moving) {
                        lds = std::max(lds, classify_lds(L->box_rows, nt));
                    }
                    ts.d[ts.n] = tn.d[tn.n] = sl->d;
                    ts.state[ts.n] = tn.state[tn.n] = state;
                    ts.level[ts.n] = tn.level[tn.n] = L->level + 1;
                    ts.start[ts.n + 1] = ts.start[ts.n] + sb;
                    tn.start[tn.n + 1] =
                        tn.start[tn.n] + parts_blocks(!moving      ? kPartsNear
                                                      : many       ? kPartsClear
                                                      : L->overlap ? kPartsSplit
                                                                   : kPartsOne,
                                                      L->np, near_wall_blocks(L->g, L->has_walls, nt));
                    ts.n++;
                    tn.n++;
                    if (ts.n == kMaxPack) {
                        int rc = flush();
                        if (rc) return rc;
                    }
                }
                int rc = flush();
                if (rc) return rc;
            }
        for (Slot *sl : act) {
            if (sl->L->tight) {
                const int rc = lbmep_step(sl->L, 1);
                if (rc) return rc;
            } else {
                advance_state(sl->L);
            }
            sl->to_enqueue -= 1;
            S->st.cell_updates += (double)sl->L->g.N;
        }
        S->st.steps += 1;
    }
    return LBMEP_OK;
}

int progress(lbmep_server *S) {
    // 1. retire slots whose read-out has completed
    for (Slot &sl : S->slots) {
        if (!sl.req || !sl.retiring) continue;
        const hipError_t q = hipEventQuery(sl.ev);
        if (q == hipErrorNotReady) continue;
        if (q != hipSuccess) return fail(LBMEP_EDEVICE, std::string("event: ") + hipGetErrorString(q));
        retire(S, sl);
    }
    // 2. drop completed chunk events
    while (!S->chunk_ev.empty()) {
        const hipError_t q = hipEventQuery(S->chunk_ev.front());
        if (q == hipErrorNotReady) break;
        if (q != hipSuccess) return fail(LBMEP_EDEVICE, std::string("event: ") + hipGetErrorString(q));
        S->ev_pool.push_back(S->chunk_ev.front());
        S->chunk_ev.pop_front();
        S->st.cell_updates_done += S->chunk_work.front();
        S->chunk_work.pop_front();
    }
    // 3. admit queued requests (FIFO) while a slot is free and the budget holds
    while (!S->queue.empty()) {
        Request *r = S->queue.front().get();
        if (S->reserved + r->footprint > S->arena.size()) break;
        Slot *free_slot = nullptr;
        for (Slot &sl : S->slots)
            if (!sl.req) {
                free_slot = &sl;
                break;
            }
        if (!free_slot) break;
        std::unique_ptr<Request> owned = std::move(S->queue.front());
        S->queue.pop_front();
        const int rc = admit(S, *free_slot, r);
        if (rc) {
            if (rc == LBMEP_ENOMEM && S->reserved > 0) {
                // fragmentation: wait for a resident request to finish
                S->queue.push_front(std::move(owned));
                break;
            }
            fail_request(r, rc, lbmep_last_error());
            r->t_admit = r->t_done = now_s(S->t0);
            r->done = true;
            S->st.failed += 1;
            S->unreported.push_back(r->id);
            S->finished[r->id] = std::move(owned);
            continue;
        }
        owned.release();  // held by the slot until it retires
        S->reserved += r->footprint;
        S->st.admitted += 1;
        if (free_slot->to_enqueue == 0) {
            int rc2 = enqueue_readout(S, *free_slot);
            if (rc2) return rc2;
        }
    }
    // 4. keep two chunks in flight
    while (S->chunk_ev.size() < 2) {
        std::vector<Slot *> act;
        int k = S->cfg.chunk_steps;
        for (Slot &sl : S->slots)
            if (sl.req && !sl.retiring && sl.to_enqueue > 0) {
                act.push_back(&sl);
                k = std::min(k, sl.to_enqueue);
            }
        if (act.empty()) break;
        const double before = S->st.cell_updates;
        int rc = enqueue_steps(S, act, k);
        if (rc) return rc;
        for (Slot *sl : act)
            if (sl->to_enqueue == 0) {
                rc = enqueue_readout(S, *sl);
                if (rc) return rc;
            }
        hipEvent_t e = get_event(S);
        if (!e) return fail(LBMEP_EDEVICE, "event creation failed");
        LBMEP_HIP_TRY(hipEventRecord(e, S->main));
        S->chunk_ev.push_back(e);
        S->chunk_work.push_back(S->st.cell_updates - before);
        S->st.chunks += 1;
    }
    return LBMEP_OK;
}

}  // namespace

extern "C" {

int lbmep_server_create(const lbmep_server_config *cfg, lbmep_server **out) {
    if (!cfg || !out) return fail(LBMEP_EINVAL, "null argument");
    *out = nullptr;
    if (cfg->max_slots < 1 || cfg->max_slots > kMaxPack)
        return fail(LBMEP_EINVAL, "max_slots must be in [1, 64]");
    if (cfg->chunk_steps < 1) return fail(LBMEP_EINVAL, "chunk_steps must be >= 1");
    if (cfg->max_queue < 1) return fail(LBMEP_EINVAL, "max_queue must be >= 1");
    if (cfg->hbm_budget < (size_t(1) << 20)) return fail(LBMEP_EINVAL, "budget below 1 MiB");
    int ndev = 0;
    LBMEP_HIP_TRY(hipGetDeviceCount(&ndev));
    if (cfg->device < 0 || cfg->device >= ndev) return fail(LBMEP_EINVAL, "no such device");
    LBMEP_HIP_TRY(hipSetDevice(cfg->device));
    auto S = std::make_unique<lbmep_server>();
    S->cfg = *cfg;
    S->t0 = std::chrono::steady_clock::now();
    if (S->arena.init(cfg->hbm_budget) != hipSuccess)
        return fail(LBMEP_ENOMEM, "device arena allocation failed");
    LBMEP_HIP_TRY(hipStreamCreateWithFlags(&S->main, hipStreamNonBlocking));
    LBMEP_HIP_TRY(hipStreamCreateWithFlags(&S->setup, hipStreamNonBlocking));
    LBMEP_HIP_TRY(hipStreamCreateWithFlags(&S->copy, hipStreamNonBlocking));
    S->pinned.set_limit(std::min(S->arena.size(), size_t(1) << 30));
    S->slots.resize(cfg->max_slots);
    S->st.budget = S->arena.size();
    *out = S.release();
    return LBMEP_OK;
}

int lbmep_server_destroy(lbmep_server *S) {
    if (!S) return LBMEP_OK;
    hipSetDevice(S->cfg.device);
    hipStreamSynchronize(S->main);
    hipStreamSynchronize(S->setup);
    hipStreamSynchronize(S->copy);
    for (Slot &sl : S->slots) {
        if (!sl.req) continue;
        S->arena.release(sl.fields);
        S->arena.release(sl.d);
        destroy_lattice(sl.L, false);
        if (sl.ev) hipEventDestroy(sl.ev);
        delete sl.req;
    }
    for (hipEvent_t e : S->chunk_ev) hipEventDestroy(e);
    for (hipEvent_t e : S->ev_pool) hipEventDestroy(e);
    hipStreamDestroy(S->main);
    hipStreamDestroy(S->setup);
    hipStreamDestroy(S->copy);
    delete S;
    return LBMEP_OK;
}

int lbmep_server_request_footprint(const lbmep_request *q, size_t *bytes) {
    if (!q || !bytes) return fail(LBMEP_EINVAL, "null argument");
    int rc = check_config(&q->cfg);
    if (rc) return rc;
    double rmax = 0.0;
    for (int i = 0; q->R && i < q->n; ++i) rmax = std::max(rmax, q->R[i]);
    *bytes = request_footprint(q->cfg, q->n, rmax, q->rho_e != nullptr, q->flags != nullptr,
                               q->keep_fields != 0, false);
    return LBMEP_OK;
}

int lbmep_server_submit(lbmep_server *S, const lbmep_request *q, uint64_t *id) {
    if (!S || !q || !id) return fail(LBMEP_EINVAL, "null argument");
    lbmep_config c = q->cfg;
    c.device = S->cfg.device;
    c.stream = nullptr;
    int rc = check_config(&c);
    if (rc) return rc;
    if (q->steps < 1) return fail(LBMEP_EINVAL, "steps must be >= 1");
    if (q->n < 0) return fail(LBMEP_EINVAL, "negative particle count");
    if (q->n > 0 && (!q->X || !q->R || !q->U)) return fail(LBMEP_EINVAL, "null particle array");
    if (q->rho_e && q->rho_e_dtype != LBMEP_DTYPE_F64 && q->rho_e_dtype != LBMEP_DTYPE_F32)
        return fail(LBMEP_EINVAL, "unknown rho_e dtype");
    if (q->rho_e && !finite_all(q->E, 3)) return fail(LBMEP_EINVAL, "bad field E");
    if (!small_offsets(c))
        return fail(LBMEP_EINVAL, "grid too large for the packed sweep (two population grids "
                                  "must be below 4 GiB)");
    const size_t N = (size_t)c.nx * c.ny * c.nz;
    double rmax = 0.0;
    for (int i = 0; i < q->n; ++i)
        if (std::isfinite(q->R[i])) rmax = std::max(rmax, q->R[i]);
    auto footprint = [&](bool tight) {
        return request_footprint(c, q->n, rmax, q->rho_e != nullptr, q->flags != nullptr,
                                 q->keep_fields != 0, tight);
    };
    size_t fp = footprint(false);
    const bool tight = fp > S->arena.size();
    if (tight) fp = footprint(true);
    if (fp > S->arena.size()) return fail(LBMEP_EINVAL, "request footprint exceeds the budget");
    if ((int32_t)S->queue.size() >= S->cfg.max_queue) return fail(LBMEP_EBUSY, "queue full");
    auto r = std::make_unique<Request>();
    r->cfg = c;
    r->n = q->n;
    r->steps = q->steps;
    if (q->flags) r->flags.assign(q->flags, q->flags + N);
    if (q->n > 0) {
        r->X.assign(q->X, q->X + 3 * (size_t)q->n);
        r->R.assign(q->R, q->R + q->n);
        r->U.assign(q->U, q->U + 3 * (size_t)q->n);
        if (q->W)
            r->W.assign(q->W, q->W + 3 * (size_t)q->n);
        else
            r->W.assign(3 * (size_t)q->n, 0.0);
    }
    if (q->rho_e) {
        const size_t b = N * (q->rho_e_dtype == LBMEP_DTYPE_F64 ? 8 : 4);
        r->rho_e.assign(static_cast<const char *>(q->rho_e), static_cast<const char *>(q->rho_e) + b);
        r->rho_dtype = q->rho_e_dtype;
        r->charge = true;
        for (int k = 0; k < 3; ++k) r->E[k] = q->E[k];
    }
    r->keep_fields = q->keep_fields != 0;
    r->footprint = fp;
    r->tight = tight;
    r->id = S->next_id++;
    r->t_submit = now_s(S->t0);
    *id = r->id;
    S->queue.push_back(std::move(r));
    S->st.submitted += 1;
    return LBMEP_OK;
}

int lbmep_server_poll(lbmep_server *S, uint64_t *done_ids, int32_t cap, int32_t *ndone) {
    if (!S || !ndone || cap < 0 || (cap > 0 && !done_ids)) return fail(LBMEP_EINVAL, "bad argument");
    LBMEP_HIP_TRY(hipSetDevice(S->cfg.device));
    *ndone = 0;
    int rc = progress(S);
    if (rc) return rc;
    while (*ndone < cap && !S->unreported.empty()) {
        done_ids[(*ndone)++] = S->unreported.front();
        S->unreported.pop_front();
    }
    return LBMEP_OK;
}

int lbmep_server_result(lbmep_server *S, uint64_t id, double *F, double *M, double inv[4],
                        double times[3]) {
    if (!S) return fail(LBMEP_EINVAL, "null server");
    auto it = S->finished.find(id);
    if (it == S->finished.end()) return fail(LBMEP_ESTATE, "request not finished (or unknown)");
    Request *r = it->second.get();
    if (r->status != LBMEP_OK) return fail(r->status, "request failed: " + r->error);
    if (F && !r->F.empty()) std::memcpy(F, r->F.data(), r->F.size() * sizeof(double));
    if (M && !r->M.empty()) std::memcpy(M, r->M.data(), r->M.size() * sizeof(double));
    if (inv) std::memcpy(inv, r->inv, sizeof r->inv);
    if (times) {
        times[0] = r->t_submit;
        times[1] = r->t_admit;
        times[2] = r->t_done;
    }
    return LBMEP_OK;
}

int lbmep_server_fields(lbmep_server *S, uint64_t id, double *rho, double *u) {
    if (!S || !rho || !u) return fail(LBMEP_EINVAL, "null argument");
    auto it = S->finished.find(id);
    if (it == S->finished.end()) return fail(LBMEP_ESTATE, "request not finished (or unknown)");
    Request *r = it->second.get();
    if (r->status != LBMEP_OK) return fail(r->status, "request failed: " + r->error);
    if (!r->keep_fields) return fail(LBMEP_ESTATE, "request was submitted without keep_fields");
    const size_t N = (size_t)r->cfg.nx * r->cfg.ny * r->cfg.nz;
    copy_out(rho, r->fields ? r->fields : r->rho.data(), N * sizeof(double));
    copy_out(u, r->fields ? r->fields + N : r->u.data(), 3 * N * sizeof(double));
    return LBMEP_OK;
}

int lbmep_server_release(lbmep_server *S, uint64_t id) {
    if (!S) return fail(LBMEP_EINVAL, "null server");
    auto it = S->finished.find(id);
    if (it == S->finished.end()) return fail(LBMEP_ESTATE, "request not finished (or unknown)");
    S->pinned.give(it->second->fields);
    S->finished.erase(it);
    return LBMEP_OK;
}

int lbmep_server_get_stats(lbmep_server *S, lbmep_server_stats *out) {
    if (!S || !out) return fail(LBMEP_EINVAL, "null argument");
    S->st.queued = (int32_t)S->queue.size();
    int32_t res = 0;
    for (const Slot &sl : S->slots) res += sl.req ? 1 : 0;
    S->st.resident = res;
    S->st.bytes_reserved = S->reserved;
    S->st.bytes_in_use = S->arena.used();
    *out = S->st;
    return LBMEP_OK;
}

int lbmep_server_now(lbmep_server *S, double *t) {
    if (!S || !t) return fail(LBMEP_EINVAL, "null argument");
    *t = now_s(S->t0);
    return LBMEP_OK;
}

}  // extern "C"
