// Host batching front-end: staging, state gather/scatter and the pipelined
// round (copy stream + compute stream).  Included at the end of seedinf.hip.
#pragma once
#include <atomic>

namespace seedinf {

// What a batch's step reads besides the frames, one block per row: the actor's recurrent state and last action, and the
// row's small inputs, which come straight from the pinned staging set (a few dozen bytes a row: copied one array at a time
// they were five transfers).  Launched before the frames have arrived.
struct BatchRows {
    // pinned host memory
    const int32_t* actor; const float* reward; const uint8_t* done; const float* uniforms; const float* epsilon; const float* explore;
    // device
    int32_t* d_actor; float* d_reward; uint8_t* d_done; float* d_uniforms; float* d_epsilon; float* d_explore;
    int32_t* d_prev_action; float* d_h_in; float* d_c_in;
    float* st_h; float* st_c; int32_t* st_action;            // per actor
    int A, Hn;
};
__global__ __launch_bounds__(256) void batch_gather_kernel(BatchRows p)
{
    const int r = blockIdx.x, tid = threadIdx.x;
    const int actor = p.actor[r];
    for (int i = tid; i < p.Hn; i += 256) {
        p.d_h_in[(size_t)r * p.Hn + i] = p.st_h[(size_t)actor * p.Hn + i];
        p.d_c_in[(size_t)r * p.Hn + i] = p.st_c[(size_t)actor * p.Hn + i];
    }
    if (p.uniforms)
        for (int i = tid; i < p.A; i += 256) p.d_uniforms[(size_t)r * p.A + i] = p.uniforms[(size_t)r * p.A + i];
    if (tid == 0) {
        p.d_actor[r] = actor;
        p.d_prev_action[r] = p.st_action[actor];
        p.d_reward[r] = p.reward[r];
        p.d_done[r] = p.done[r];
        if (p.epsilon) p.d_epsilon[r] = p.epsilon[r];
    }
    if (p.epsilon && tid < 2) p.d_explore[2 * r + tid] = p.explore[2 * r + tid];
}

// The step's new states and actions back to their actors, and the actions to pinned host memory.
__global__ __launch_bounds__(256) void batch_scatter_kernel(BatchRows p, const float* __restrict__ h_out, const float* __restrict__ c_out,
                                                            const int32_t* __restrict__ actions, int32_t* __restrict__ actions_host)
{
    const int r = blockIdx.x, tid = threadIdx.x;
    const int actor = p.d_actor[r];
    for (int i = tid; i < p.Hn; i += 256) {
        p.st_h[(size_t)actor * p.Hn + i] = h_out[(size_t)r * p.Hn + i];
        p.st_c[(size_t)actor * p.Hn + i] = c_out[(size_t)r * p.Hn + i];
    }
    if (tid == 0) {
        const int a = actions[r];
        p.st_action[actor] = a;
        actions_host[r] = a;
    }
}

}  // namespace seedinf

constexpr int BATCHER_CHUNKS = 8;

struct seed_batcher {
    seed_infer* h = nullptr;
    int n_actors = 0, max_rows = 0, A = 0, Hn = 0;
    size_t frame = 0;
    int chunk = 0;                      // rows whose torso starts together while later frames travel
    hipStream_t copy_s = nullptr, comp_s = nullptr;
    // per-actor device state
    float* st_h = nullptr; float* st_c = nullptr; int32_t* st_action = nullptr;
    struct Set {
        // pinned host staging
        uint8_t* obs = nullptr; float* reward = nullptr; uint8_t* done = nullptr; int32_t* actor = nullptr;
        float* uniforms = nullptr; float* epsilon = nullptr; float* explore = nullptr; int32_t* actions = nullptr;
        // device mirrors and per-batch work buffers
        uint8_t* d_obs = nullptr; float* d_reward = nullptr; uint8_t* d_done = nullptr; int32_t* d_actor = nullptr;
        float* d_uniforms = nullptr; float* d_epsilon = nullptr; float* d_explore = nullptr;
        int32_t* d_prev_action = nullptr; int32_t* d_actions = nullptr;
        float* d_h_in = nullptr; float* d_c_in = nullptr; float* d_h_out = nullptr; float* d_c_out = nullptr;
        float* d_logits = nullptr; float* d_value = nullptr;
        hipEvent_t ready[BATCHER_CHUNKS] = {};   // the frames of the first there[k] rows have arrived; the last in use: all
        int there[BATCHER_CHUNKS] = {};
        hipEvent_t finished = nullptr;
        int chunks = 0;                 // of `ready` recorded
        int marked = 0;                 // rows sent when the last of them was (before the submit)
        int rows = 0;                   // rows added to the batch being filled
        int sent = 0;                   // leading rows whose frames are on their way to the device
        bool open = false;              // a row was reserved: its frame may be written until submit
        int result_rows = 0;            // rows of the submitted batch `ticket`
        int ticket = -1;
        bool in_flight = false;
    } set[2];
    int fill = 0;                       // staging set being filled
    int next_ticket = 0;
    std::vector<int32_t> seen;          // per actor: ticket of the batch it was last added to
    std::string err;
};

#define B_TRY(b, expr)                                                                \
    do {                                                                              \
        hipError_t e_ = (expr);                                                       \
        if (e_ != hipSuccess) {                                                       \
            (b)->err = std::string(#expr) + ": " + hipGetErrorString(e_);             \
            return e_ == hipErrorOutOfMemory ? SEED_ERR_OOM : SEED_ERR_DEVICE;        \
        }                                                                             \
    } while (0)

static void batcher_free(seed_batcher* b)
{
    if (!b) return;
    if (b->comp_s) (void)hipStreamSynchronize(b->comp_s);
    if (b->copy_s) (void)hipStreamSynchronize(b->copy_s);
    for (auto& s : b->set) {
        void* host[] = {s.obs, s.reward, s.done, s.actor, s.uniforms, s.epsilon, s.explore, s.actions};
        for (void* p : host) if (p) (void)hipHostFree(p);
        void* dev[] = {s.d_obs, s.d_reward, s.d_done, s.d_actor, s.d_uniforms, s.d_epsilon, s.d_explore, s.d_prev_action,
                       s.d_actions, s.d_h_in, s.d_c_in, s.d_h_out, s.d_c_out, s.d_logits, s.d_value};
        for (void* p : dev) if (p) (void)hipFree(p);
        for (hipEvent_t e : s.ready) if (e) (void)hipEventDestroy(e);
        if (s.finished) (void)hipEventDestroy(s.finished);
    }
    if (b->st_h) (void)hipFree(b->st_h);
    if (b->st_c) (void)hipFree(b->st_c);
    if (b->st_action) (void)hipFree(b->st_action);
    if (b->copy_s) (void)hipStreamDestroy(b->copy_s);
    if (b->comp_s) (void)hipStreamDestroy(b->comp_s);
    delete b;
}

static seed_status_t batcher_alloc(seed_batcher* b)
{
    const size_t R = (size_t)b->max_rows, A = (size_t)b->A, Hn = (size_t)b->Hn, N = (size_t)b->n_actors;
    B_TRY(b, hipStreamCreateWithFlags(&b->copy_s, hipStreamNonBlocking));
    B_TRY(b, hipStreamCreateWithFlags(&b->comp_s, hipStreamNonBlocking));
    B_TRY(b, hipMalloc(&b->st_action, N * sizeof(int32_t)));
    B_TRY(b, hipMemset(b->st_action, 0, N * sizeof(int32_t)));
    if (Hn) {
        B_TRY(b, hipMalloc(&b->st_h, N * Hn * sizeof(float)));
        B_TRY(b, hipMalloc(&b->st_c, N * Hn * sizeof(float)));
        B_TRY(b, hipMemset(b->st_h, 0, N * Hn * sizeof(float)));
        B_TRY(b, hipMemset(b->st_c, 0, N * Hn * sizeof(float)));
    }
    for (auto& s : b->set) {
        B_TRY(b, hipHostMalloc((void**)&s.obs, R * b->frame, hipHostMallocDefault));
        B_TRY(b, hipHostMalloc((void**)&s.reward, R * sizeof(float), hipHostMallocDefault));
        B_TRY(b, hipHostMalloc((void**)&s.done, R, hipHostMallocDefault));
        B_TRY(b, hipHostMalloc((void**)&s.actor, R * sizeof(int32_t), hipHostMallocDefault));
        B_TRY(b, hipHostMalloc((void**)&s.uniforms, R * A * sizeof(float), hipHostMallocDefault));
        B_TRY(b, hipHostMalloc((void**)&s.epsilon, R * sizeof(float), hipHostMallocDefault));
        B_TRY(b, hipHostMalloc((void**)&s.explore, R * 2 * sizeof(float), hipHostMallocDefault));
        B_TRY(b, hipHostMalloc((void**)&s.actions, R * sizeof(int32_t), hipHostMallocDefault));
        B_TRY(b, hipMalloc(&s.d_obs, R * b->frame));
        B_TRY(b, hipMalloc(&s.d_reward, R * sizeof(float)));
        B_TRY(b, hipMalloc(&s.d_done, R));
        B_TRY(b, hipMalloc(&s.d_actor, R * sizeof(int32_t)));
        B_TRY(b, hipMalloc(&s.d_uniforms, R * A * sizeof(float)));
        B_TRY(b, hipMalloc(&s.d_epsilon, R * sizeof(float)));
        B_TRY(b, hipMalloc(&s.d_explore, R * 2 * sizeof(float)));
        B_TRY(b, hipMalloc(&s.d_prev_action, R * sizeof(int32_t)));
        B_TRY(b, hipMalloc(&s.d_actions, R * sizeof(int32_t)));
        B_TRY(b, hipMalloc(&s.d_logits, R * A * sizeof(float)));
        B_TRY(b, hipMalloc(&s.d_value, R * sizeof(float)));
        if (Hn) {
            B_TRY(b, hipMalloc(&s.d_h_in, R * Hn * sizeof(float)));
            B_TRY(b, hipMalloc(&s.d_c_in, R * Hn * sizeof(float)));
            B_TRY(b, hipMalloc(&s.d_h_out, R * Hn * sizeof(float)));
            B_TRY(b, hipMalloc(&s.d_c_out, R * Hn * sizeof(float)));
        }
        for (hipEvent_t& e : s.ready) B_TRY(b, hipEventCreateWithFlags(&e, hipEventDisableTiming));
        B_TRY(b, hipEventCreateWithFlags(&s.finished, hipEventDisableTiming));
    }
    B_TRY(b, hipDeviceSynchronize());
    return SEED_OK;
}

extern "C" seed_status_t seed_batcher_create(seed_infer_t* h, int32_t n_actors, seed_batcher_t** out)
{
    g_create_err.clear();
    if (!h || !out) { g_create_err = "handle or out is NULL"; return SEED_ERR_INVALID_ARG; }
    if (n_actors <= 0 || n_actors > (1 << 24)) { g_create_err = "n_actors must be in 1..2^24"; return SEED_ERR_INVALID_ARG; }
    seed_batcher* b = new (std::nothrow) seed_batcher;
    if (!b) { g_create_err = "host allocation failed"; return SEED_ERR_OOM; }
    const seed_arch_t& a = h->plan.arch;
    b->h = h; b->n_actors = n_actors; b->max_rows = a.max_batch; b->A = a.num_actions; b->Hn = a.lstm_units;
    b->frame = (size_t)a.obs_h * a.obs_w * a.obs_c;
    b->seen.assign((size_t)n_actors, -1);
    // whole rounds of the torso over the compute units, at most BATCHER_CHUNKS of them
    int n_cu = 0;
    if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, h->device) != hipSuccess || n_cu <= 0) n_cu = 256;
    b->chunk = ((a.max_batch + BATCHER_CHUNKS - 1) / BATCHER_CHUNKS + n_cu - 1) / n_cu * n_cu;
    seed_status_t st = batcher_alloc(b);
    if (st != SEED_OK) { g_create_err = b->err; batcher_free(b); return st; }
    *out = b;
    return SEED_OK;
}

extern "C" void seed_batcher_destroy(seed_batcher_t* b) { batcher_free(b); }
extern "C" const char* seed_batcher_last_error(const seed_batcher_t* b) { return b ? b->err.c_str() : g_create_err.c_str(); }
extern "C" void* seed_batcher_stream(seed_batcher_t* b) { return b ? (void*)b->comp_s : nullptr; }

// Frames travel while later rows are still being added, in transfers of at least this many bytes (each costs about 9 us more;
// a round of 512 DMLab frames is 10.6 MB, 193 us of PCIe in one transfer), unless another batch is in flight: then the link is busy
// with that batch's frames or the device with its step, cutting this one's frames up only adds the 9 us, and they
// go in one transfer at the submit.  Without early transfers, with them always, now, us a round: 512 DMLab frames alone
// 431, -, 356 (left is the copy to pinned memory, 260 us where neither side of it is in cache; stores past the
// caches or items handed out to whichever thread is awake made it no shorter); two in flight, 1024 Football frames 2138, 2320,
// 2119, 1024 Atari frames 559, 615, 540, 4096 DMLab frames 1949, 1930, 1830.
constexpr size_t BATCHER_SEND_BYTES = (size_t)1 << 21;

// Starts the transfer of the filled rows [sent, rows).
static seed_status_t batcher_copy(seed_batcher* b, seed_batcher::Set& s, int rows)
{
    const size_t from = (size_t)s.sent * b->frame, bytes = (size_t)(rows - s.sent) * b->frame;
    if (bytes) B_TRY(b, hipMemcpyAsync(s.d_obs + from, s.obs + from, bytes, hipMemcpyHostToDevice, b->copy_s));
    s.sent = rows;
    return SEED_OK;
}

// Event k: the leading `rows` rows have arrived once what was sent so far has.
static seed_status_t batcher_mark(seed_batcher* b, seed_batcher::Set& s, int k, int rows)
{
    B_TRY(b, hipEventRecord(s.ready[k], b->copy_s));
    s.there[k] = rows;
    return SEED_OK;
}

// A transfer before the submit, if the rows are worth one, and an event for the whole chunks that it completes (the last
// event is the submit's).
static seed_status_t batcher_send(seed_batcher* b, seed_batcher::Set& s, int rows)
{
    if (b->set[b->fill ^ 1].in_flight || (size_t)(rows - s.sent) * b->frame < BATCHER_SEND_BYTES) return SEED_OK;
    if (seed_status_t st = batcher_copy(b, s, rows); st != SEED_OK) return st;
    const int whole = rows / b->chunk * b->chunk, marked = s.chunks ? s.there[s.chunks - 1] : 0;
    if (whole <= marked || s.chunks >= BATCHER_CHUNKS - 1) return SEED_OK;
    if (seed_status_t st = batcher_mark(b, s, s.chunks, whole); st != SEED_OK) return st;
    ++s.chunks;
    s.marked = rows;
    return SEED_OK;
}

static seed_status_t batcher_row(seed_batcher* b, int32_t actor, float prev_reward, uint8_t done, uint8_t** obs_slot)
{
    auto fail = [&](seed_status_t st, const char* m) { b->err = m; return st; };
    if (actor < 0 || actor >= b->n_actors) return fail(SEED_ERR_INVALID_ARG, "actor out of range");
    seed_batcher::Set& s = b->set[b->fill];
    if (s.in_flight) {
        // this staging set's earlier batch must have left the host buffers before they are overwritten
        B_TRY(b, hipEventSynchronize(s.finished));
        s.in_flight = false;
        s.rows = s.sent = s.chunks = 0;
        s.open = false;
        s.ticket = -1;                  // its results were never collected and are about to be overwritten
    }
    if (s.rows >= b->max_rows) return fail(SEED_ERR_BATCH_TOO_LARGE, "the batch already holds max_batch rows");
    if (b->seen[actor] == b->next_ticket) return fail(SEED_ERR_INVALID_ARG, "actor added twice to one batch");
    b->seen[actor] = b->next_ticket;
    const int r = s.rows++;
    s.reward[r] = prev_reward;
    s.done[r] = done;
    s.actor[r] = actor;
    *obs_slot = s.obs + (size_t)r * b->frame;
    return SEED_OK;
}

extern "C" seed_status_t seed_batcher_reserve(seed_batcher_t* b, int32_t actor, float prev_reward, uint8_t done,
                                              uint8_t** obs_slot)
{
    if (!b) return SEED_ERR_INVALID_ARG;
    if (!obs_slot) { b->err = "obs_slot is NULL"; return SEED_ERR_INVALID_ARG; }
    const seed_status_t st = batcher_row(b, actor, prev_reward, done, obs_slot);
    if (st == SEED_OK) b->set[b->fill].open = true;
    return st;
}

extern "C" seed_status_t seed_batcher_add(seed_batcher_t* b, int32_t actor, const uint8_t* obs_host, float prev_reward,
                                          uint8_t done)
{
    if (!b) return SEED_ERR_INVALID_ARG;
    if (!obs_host) { b->err = "obs_host is NULL"; return SEED_ERR_INVALID_ARG; }
    uint8_t* slot = nullptr;
    seed_status_t st = batcher_row(b, actor, prev_reward, done, &slot);
    if (st != SEED_OK) return st;
    memcpy(slot, obs_host, b->frame);
    seed_batcher::Set& s = b->set[b->fill];
    return s.open ? SEED_OK : batcher_send(b, s, s.rows);
}

extern "C" seed_status_t seed_batcher_add_many(seed_batcher_t* b, int32_t n, const int32_t* actors, const uint8_t* obs_host,
                                               const float* prev_rewards, const uint8_t* dones)
{
    if (!b) return SEED_ERR_INVALID_ARG;
    if (n < 0 || !actors || !obs_host || !prev_rewards || !dones) { b->err = "n is negative or a pointer is NULL"; return SEED_ERR_INVALID_ARG; }
    int32_t ok = 0;
    uint8_t* slot = nullptr;
    seed_status_t st = SEED_OK;
    for (; ok < n; ++ok) {
        st = batcher_row(b, actors[ok], prev_rewards[ok], dones[ok], &slot);
        if (st != SEED_OK) break;
    }
    if (ok == 0) return st;
    // The frame copies are the expensive part: from about a megabyte on they go over the handle's persistent host threads
    // (below, waking them costs more than it saves: 512 DMLab frames in groups of 32, 0.66 MB, 528 us a round on the calling
    // thread, 673 on three), in pieces of about a quarter of a megabyte, and the calling thread sends on whatever is
    // complete from the front after each piece of its own.
    seed_batcher::Set& s = b->set[b->fill];
    const int32_t first = s.rows - ok;
    const int32_t per = (int32_t)std::max<size_t>(1, ((size_t)1 << 18) / b->frame);
    const int pieces = (ok + per - 1) / per;
    HostPool* pool = (size_t)ok * b->frame > (size_t)1 << 20 && pieces > 1 ? host_pool(b->h) : nullptr;
    std::vector<std::atomic<uint8_t>> copied((size_t)pieces);
    for (auto& c : copied) c.store(0, std::memory_order_relaxed);
    int front = 0;                                           // pieces complete from the front
    seed_status_t sent = SEED_OK;
    const std::thread::id caller = std::this_thread::get_id();
    auto copy = [&](int t) {
        const int32_t i0 = t * per, i1 = std::min(ok, i0 + per);
        memcpy(s.obs + (size_t)(first + i0) * b->frame, obs_host + (size_t)i0 * b->frame, (size_t)(i1 - i0) * b->frame);
        copied[t].store(1, std::memory_order_release);
        if (s.open || std::this_thread::get_id() != caller || sent != SEED_OK) return;      // (`front` and `sent` are the caller's)
        while (front < pieces && copied[front].load(std::memory_order_acquire)) ++front;
        sent = batcher_send(b, s, first + std::min(ok, front * per));
    };
    if (pool) pool->run(pieces, copy);
    else for (int t = 0; t < pieces; ++t) copy(t);
    if (!s.open && sent == SEED_OK) sent = batcher_send(b, s, s.rows);
    return st != SEED_OK ? st : sent;
}

extern "C" seed_status_t seed_batcher_submit(seed_batcher_t* b, const float* uniforms_host, const float* epsilon_host,
                                             const float* explore_host, int32_t* ticket)
{
    if (!b || !ticket) return SEED_ERR_INVALID_ARG;
    auto fail = [&](seed_status_t st, const char* m) { b->err = m; return st; };
    seed_batcher::Set& s = b->set[b->fill];
    const seed_arch_t& a = b->h->plan.arch;
    const int R = s.in_flight ? 0 : s.rows;                  // (in flight: the rows are the unfinished batch's)
    if (R == 0) return fail(SEED_ERR_INVALID_ARG, "the batch is empty");
    if (a.select == SEED_SELECT_GUMBEL && !uniforms_host) return fail(SEED_ERR_INVALID_ARG, "Gumbel-max selection needs uniforms");
    if (a.select == SEED_SELECT_GREEDY && uniforms_host) return fail(SEED_ERR_INVALID_ARG, "greedy selection takes no uniforms (pass NULL)");
    if ((epsilon_host == nullptr) != (explore_host == nullptr)) return fail(SEED_ERR_INVALID_ARG, "epsilon and explore_uniforms must be given together");
    // (before anything is enqueued: a copy or launch that went ahead would stand when the step is refused)
    int dev = -1;
    B_TRY(b, hipGetDevice(&dev));
    if (dev != b->h->device) return fail(SEED_ERR_INVALID_ARG, "current HIP device differs from the handle's device");
    const size_t A = (size_t)b->A, Hn = (size_t)b->Hn;
    if (uniforms_host) memcpy(s.uniforms, uniforms_host, R * A * sizeof(float));
    if (epsilon_host) {
        memcpy(s.epsilon, epsilon_host, R * sizeof(float));
        memcpy(s.explore, explore_host, R * 2 * sizeof(float));
    }
    // the frames not yet sent, on the copy stream (overlaps the previous batch's compute); beside them, on the compute
    // stream, the rows' states and small inputs; the step waits for both
    hipStream_t ks = b->comp_s;
    const bool rec = Hn > 0;
    if (seed_status_t st = batcher_copy(b, s, R); st != SEED_OK) return st;
    // one more event for the rows behind the last one's, unless that one came behind the last transfer
    int events = s.chunks;
    if (events > 0 && s.marked == R) s.there[events - 1] = R;
    else if (seed_status_t st = batcher_mark(b, s, events++, R); st != SEED_OK) return st;
    const FrameArrival arrival{events, s.there, s.ready};
    BatchRows br{};
    br.actor = s.actor; br.reward = s.reward; br.done = s.done;
    br.uniforms = uniforms_host ? s.uniforms : nullptr;
    br.epsilon = epsilon_host ? s.epsilon : nullptr; br.explore = s.explore;
    br.d_actor = s.d_actor; br.d_reward = s.d_reward; br.d_done = s.d_done; br.d_uniforms = s.d_uniforms; br.d_epsilon = s.d_epsilon; br.d_explore = s.d_explore;
    br.d_prev_action = s.d_prev_action; br.d_h_in = s.d_h_in; br.d_c_in = s.d_c_in;
    br.st_h = b->st_h; br.st_c = b->st_c; br.st_action = b->st_action; br.A = (int)A; br.Hn = (int)Hn;
    hipLaunchKernelGGL(batch_gather_kernel, dim3(R), dim3(256), 0, ks, br);
    seed_step_ext_t ext{};
    ext.struct_size = sizeof(ext);
    ext.done = rec ? s.d_done : nullptr;
    ext.epsilon = epsilon_host ? s.d_epsilon : nullptr;
    ext.explore_uniforms = epsilon_host ? s.d_explore : nullptr;
    seed_status_t st = step_impl(b->h, R, s.d_obs, rec ? s.d_prev_action : nullptr, rec ? s.d_reward : nullptr,
                                           rec ? s.d_h_in : nullptr, rec ? s.d_c_in : nullptr,
                                           uniforms_host ? s.d_uniforms : nullptr, &ext, s.d_actions, s.d_logits, s.d_value,
                                           rec ? s.d_h_out : nullptr, rec ? s.d_c_out : nullptr, nullptr, ks, false, &arrival);
    if (st != SEED_OK) { b->err = b->h->err; return st; }
    hipLaunchKernelGGL(batch_scatter_kernel, dim3(R), dim3(256), 0, ks, br, s.d_h_out, s.d_c_out, s.d_actions, s.actions);
    B_TRY(b, hipEventRecord(s.finished, ks));
    B_TRY(b, hipGetLastError());
    s.ticket = b->next_ticket;
    s.result_rows = R;
    s.in_flight = true;
    *ticket = b->next_ticket++;
    b->fill ^= 1;
    // the set that is filled next starts empty; if its own batch is still in flight the first add waits for it
    seed_batcher::Set& n = b->set[b->fill];
    if (!n.in_flight) { n.rows = n.sent = n.chunks = 0; n.open = false; }
    return SEED_OK;
}

extern "C" seed_status_t seed_batcher_wait(seed_batcher_t* b, int32_t ticket, int32_t* actions_out, int32_t capacity,
                                           int32_t* n_rows)
{
    if (!b || !actions_out || !n_rows) return SEED_ERR_INVALID_ARG;
    auto fail = [&](seed_status_t st, const char* m) { b->err = m; return st; };
    for (auto& s : b->set) {
        if (s.ticket != ticket) continue;
        if (capacity < s.result_rows) return fail(SEED_ERR_INVALID_ARG, "actions_out is too small");
        B_TRY(b, hipEventSynchronize(s.finished));
        memcpy(actions_out, s.actions, (size_t)s.result_rows * sizeof(int32_t));
        *n_rows = s.result_rows;
        if (s.in_flight) {              // finished: the set may be refilled
            s.in_flight = false;
            s.rows = s.sent = s.chunks = 0;
            s.open = false;
        }
        return SEED_OK;
    }
    return fail(SEED_ERR_INVALID_ARG, "unknown ticket (only the two most recent batches can be waited for)");
}

extern "C" seed_status_t seed_batcher_read_state(seed_batcher_t* b, int32_t actor, float* h_host, float* c_host)
{
    if (!b || !h_host || !c_host) return SEED_ERR_INVALID_ARG;
    auto fail = [&](seed_status_t st, const char* m) { b->err = m; return st; };
    if (b->Hn == 0) return fail(SEED_ERR_INVALID_ARG, "a feed-forward arch has no recurrent state");
    if (actor < 0 || actor >= b->n_actors) return fail(SEED_ERR_INVALID_ARG, "actor out of range");
    B_TRY(b, hipStreamSynchronize(b->comp_s));
    const size_t nb = (size_t)b->Hn * sizeof(float);
    B_TRY(b, hipMemcpy(h_host, b->st_h + (size_t)actor * b->Hn, nb, hipMemcpyDeviceToHost));
    B_TRY(b, hipMemcpy(c_host, b->st_c + (size_t)actor * b->Hn, nb, hipMemcpyDeviceToHost));
    return SEED_OK;
}
