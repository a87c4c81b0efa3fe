// Host side: per-plan device state, profiling brackets, launch helpers.
// Part of pk_device.hip: included there, in this order, inside its anonymous namespace.

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct DeviceState {
    int device = -1;
    int n_cus = 256;                      // compute units of the device
    void* blob = nullptr;
    FieldMeta* fmeta = nullptr;
    PackMeta* pmeta = nullptr;
    int32_t* slot_field = nullptr;
    uint64_t* small_desc = nullptr;       // look-back descriptors of the one-launch forward pass (zero between calls)
    int32_t* small_done = nullptr;        // ... and its count of blocks that are through their look-back
    SmallSlice* small_slices[kSmallCuts] = {};   // the cuts of the one-launch forward pass
    int2* slot_info = nullptr;            // per slot (over all packs): its field, the field's table in the table list
    TableField* tfields = nullptr;        // the table field list with what the slice blocks need of a field
    TableMeta* sort_tables = nullptr;
    SlotMeta* slot_meta = nullptr;        // per (pack, slot): what the inverse kernel needs of the slot's table
    // Side streams: packs (and the pooling of a pack vs the dedup chain) are independent
    // pieces of memory-bound work; running them side by side hides launch gaps and
    // latency tails (the interleaving of packed operations of Sec. III-C, on one GPU).
    static constexpr int kSide = 8;
    hipStream_t side[kSide] = {};
    hipEvent_t ev_fork = nullptr;
    hipEvent_t ev_join[kSide] = {};
    bool overlap = true;
    std::vector<int64_t> hh_n_hot;        // HybridHash: rows in each pack's Hot-storage
    // profiling
    bool prof_on = false;
    std::vector<hipEvent_t> events;
    size_t events_used = 0;
    struct Rec { const char* name; size_t e0; };
    std::vector<Rec> recs;
};

std::string hip_msg(const char* what, hipError_t e)
{
    return std::string(what) + ": " + hipGetErrorString(e);
}

// The plan's device-side metadata as host arrays, and where each array goes inside one block of
// device memory (256-byte aligned pieces): look-back descriptors and their counter first.
struct MetaImage {
    std::vector<FieldMeta> fm;
    std::vector<PackMeta> pmv;
    std::vector<TableField> tfi;
    std::vector<SlotMeta> slm;
    std::vector<int2> sli;
    size_t o_desc, o_done, o_fm, o_pm, o_slot, o_sli, o_ss[kSmallCuts], o_tfi, o_tab, o_slm, total;
    size_t cuts;                 // bytes of the slice lists
};

void build_meta_image(const pk_plan* plan, MetaImage* mi)
{
    const size_t F = plan->fields.size(), P = plan->packs.size();
    mi->fm.resize(F);
    for (size_t f = 0; f < F; ++f) {
        const int32_t t = plan->fields[f].table;
        mi->fm[f].base_row = (uint32_t)plan->table_base[t];
        mi->fm[f].rows = (uint32_t)plan->tables[t].rows;
        mi->fm[f].col = (int32_t)plan->field_col[f];
        mi->fm[f].pack = plan->field_pack[f];
        mi->fm[f].slot = plan->field_slot[f];
        mi->fm[f].pool = plan->fields[f].pool;
        mi->fm[f].stable = -1;
        mi->fm[f].pad = 0;
        mi->fm[f].magic = ~(uint64_t)0 / (uint64_t)plan->tables[t].rows;
    }
    for (size_t i = 0; i < plan->sort_tables.size(); ++i)
        for (int32_t j = plan->sort_tables[i].field_begin; j < plan->sort_tables[i].field_end; ++j)
            mi->fm[plan->table_fields[j]].stable = (int32_t)i;
    mi->pmv.resize(P);
    for (size_t p = 0; p < P; ++p) {
        const Pack& k = plan->packs[p];
        mi->pmv[p].dim = k.dim; mi->pmv[p].dtype = k.dtype; mi->pmv[p].n_fields = (int32_t)k.fields.size();
        mi->pmv[p].first_slot = k.first_slot; mi->pmv[p].has_mean = k.has_mean ? 1 : 0;
        mi->pmv[p].first_stable = k.first_stable; mi->pmv[p].n_stables = k.n_stables; mi->pmv[p].pad = 0;
    }
    mi->tfi.resize(plan->table_fields.size());
    for (size_t i = 0; i < mi->tfi.size(); ++i) {
        const int32_t f = plan->table_fields[i];
        mi->tfi[i] = TableField{f, plan->field_slot[f], (int32_t)plan->field_col[f], plan->fields[f].pool};
    }
    mi->slm.resize(F);
    for (size_t j = 0; j < F; ++j) {
        const FieldMeta& m = mi->fm[plan->slot_field[j]];
        const TableMeta& tm = plan->sort_tables[m.stable];
        mi->slm[j] = SlotMeta{tm.key_lo, tm.word_base, tm.rows, m.pack};
    }
    mi->sli.resize(F);
    for (size_t j = 0; j < F; ++j) mi->sli[j] = make_int2(plan->slot_field[j], mi->fm[plan->slot_field[j]].stable);
    auto pad = [](size_t b) { return (b + 255) / 256 * 256; };
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += pad(bytes); return o; };
    mi->o_desc = take(((size_t)kSmallSlicesMax + kSmallSlicesMax / kDescGroup + 4096 + 2) * 8);   // per slice, then per group
    mi->o_done = take(256);
    mi->o_fm   = take(F * sizeof(FieldMeta));
    mi->o_pm   = take(P * sizeof(PackMeta));
    mi->o_slot = take(F * 4);
    mi->o_sli  = take(F * sizeof(int2));
    for (int c = 0; c < kSmallCuts; ++c) mi->o_ss[c] = take(plan->small_slices[c].size() * sizeof(SmallSlice));
    mi->cuts   = off - mi->o_ss[0];
    mi->o_tfi  = take(mi->tfi.size() * sizeof(TableField));
    mi->o_tab  = take(plan->sort_tables.size() * sizeof(TableMeta));
    mi->o_slm  = take(F * sizeof(SlotMeta));
    mi->total = off;
}

void point_into(DeviceState* ds, char* base, const MetaImage& mi)
{
    ds->small_desc = reinterpret_cast<uint64_t*>(base + mi.o_desc);
    ds->small_done = reinterpret_cast<int32_t*>(base + mi.o_done);
    ds->fmeta = reinterpret_cast<FieldMeta*>(base + mi.o_fm);
    ds->pmeta = reinterpret_cast<PackMeta*>(base + mi.o_pm);
    ds->slot_field = reinterpret_cast<int32_t*>(base + mi.o_slot);
    ds->slot_info = reinterpret_cast<int2*>(base + mi.o_sli);
    for (int c = 0; c < kSmallCuts; ++c) ds->small_slices[c] = reinterpret_cast<SmallSlice*>(base + mi.o_ss[c]);
    ds->tfields = reinterpret_cast<TableField*>(base + mi.o_tfi);
    ds->sort_tables = reinterpret_cast<TableMeta*>(base + mi.o_tab);
    ds->slot_meta = reinterpret_cast<SlotMeta*>(base + mi.o_slm);
}

// the pieces of the image that hold data (the descriptors and their counter only have to be zero)
template <typename Fn>
void for_meta_pieces(const pk_plan* plan, const MetaImage& mi, Fn&& fn)
{
    fn(mi.o_fm, mi.fm.data(), mi.fm.size() * sizeof(FieldMeta));
    fn(mi.o_pm, mi.pmv.data(), mi.pmv.size() * sizeof(PackMeta));
    fn(mi.o_slot, plan->slot_field.data(), plan->slot_field.size() * 4);
    fn(mi.o_sli, mi.sli.data(), mi.sli.size() * sizeof(int2));
    for (int c = 0; c < kSmallCuts; ++c) fn(mi.o_ss[c], plan->small_slices[c].data(), plan->small_slices[c].size() * sizeof(SmallSlice));
    fn(mi.o_tfi, mi.tfi.data(), mi.tfi.size() * sizeof(TableField));
    fn(mi.o_tab, plan->sort_tables.data(), plan->sort_tables.size() * sizeof(TableMeta));
    fn(mi.o_slm, mi.slm.data(), mi.slm.size() * sizeof(SlotMeta));
}

pk_status ensure_device_state(const pk_plan* cplan, DeviceState** out)
{
    pk_plan* plan = const_cast<pk_plan*>(cplan);
    static std::mutex create_mu;
    std::lock_guard<std::mutex> lock(create_mu);
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(PK_EHIP, hip_msg("hipGetDevice", e));
    DeviceState* ds = static_cast<DeviceState*>(plan->device_state);
    if (ds && ds->device == dev) { *out = ds; return PK_OK; }
    if (ds) return fail(PK_EINVAL, "a plan can be used on one device only");
    ds = new DeviceState();
    ds->device = dev;
    if (hipDeviceGetAttribute(&ds->n_cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ds->n_cus <= 0) ds->n_cus = 256;
    MetaImage mi;
    build_meta_image(plan, &mi);
    e = hipMalloc(&ds->blob, mi.total);
    if (e != hipSuccess) { delete ds; return fail(PK_EHIP, hip_msg("hipMalloc(plan metadata)", e)); }
    char* base = static_cast<char*>(ds->blob);
    point_into(ds, base, mi);
    // one copy for everything (a copy of its own for each of the pieces made a plan's first pass 70 us
    // longer); the descriptors and their counter start at zero
    std::vector<char> image(mi.total, 0);
    for_meta_pieces(plan, mi, [&](size_t off, const void* src, size_t bytes) {
        if (bytes) std::memcpy(image.data() + off, src, bytes);
    });
    e = hipMemcpy(base, image.data(), mi.total, hipMemcpyHostToDevice);
    if (e != hipSuccess) { (void)hipFree(ds->blob); delete ds; return fail(PK_EHIP, hip_msg("hipMemcpy(plan metadata)", e)); }
    for (int i = 0; i < DeviceState::kSide && e == hipSuccess; ++i) {
        e = hipStreamCreateWithFlags(&ds->side[i], hipStreamNonBlocking);     // default priority
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ds->ev_join[i], hipEventDisableTiming);
    }
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ds->ev_fork, hipEventDisableTiming);
    if (e != hipSuccess) { (void)hipFree(ds->blob); delete ds; return fail(PK_EHIP, hip_msg("side stream setup", e)); }
    if (plan->opts.debug & 1) ds->overlap = false;
    plan->device_state = ds;
    *out = ds;
    return PK_OK;
}

// fork: side streams wait for what the caller's stream has enqueued so far
pk_status fork_streams(DeviceState* ds, hipStream_t main, int n, int first = 0)
{
    hipError_t e = hipEventRecord(ds->ev_fork, main);
    for (int i = first; i < first + n && e == hipSuccess; ++i) e = hipStreamWaitEvent(ds->side[i], ds->ev_fork, 0);
    return e == hipSuccess ? PK_OK : fail(PK_EHIP, hip_msg("stream fork", e));
}

// join: the caller's stream waits for everything enqueued on the side streams
pk_status join_streams(DeviceState* ds, hipStream_t main, int n, int first = 0)
{
    hipError_t e = hipSuccess;
    for (int i = first; i < first + n && e == hipSuccess; ++i) {
        e = hipEventRecord(ds->ev_join[i], ds->side[i]);
        if (e == hipSuccess) e = hipStreamWaitEvent(main, ds->ev_join[i], 0);
    }
    return e == hipSuccess ? PK_OK : fail(PK_EHIP, hip_msg("stream join", e));
}

void prof_begin(DeviceState* ds, const char* name, hipStream_t s)
{
    if (!ds->prof_on) return;
    if (ds->events_used + 2 > ds->events.size()) {
        const size_t old = ds->events.size();
        ds->events.resize(old + 512);
        for (size_t i = old; i < ds->events.size(); ++i) (void)hipEventCreate(&ds->events[i]);
    }
    ds->recs.push_back({name, ds->events_used});
    (void)hipEventRecord(ds->events[ds->events_used], s);
}

void prof_end(DeviceState* ds, hipStream_t s)
{
    if (!ds->prof_on) return;
    (void)hipEventRecord(ds->events[ds->events_used + 1], s);
    ds->events_used += 2;
}

#define PK_LAUNCH(name, kernel, grid, block, shmem, ...)                                        \
    do {                                                                                        \
        prof_begin(ds, name, stream);                                                           \
        kernel<<<grid, block, shmem, stream>>>(__VA_ARGS__);                                    \
        prof_end(ds, stream);                                                                   \
        hipError_t e_ = hipGetLastError();                                                      \
        if (e_ != hipSuccess) return fail(PK_EHIP, hip_msg("launch of " name, e_));             \
    } while (0)

unsigned blocks_for(int64_t items, int64_t per_block, int64_t cap)
{
    int64_t b = (items + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

// log2 of the lanes that hold a row, four columns each
int lane_shift(int D) { int s = 0; while ((4 << s) < D) ++s; return s; }

// pack p's packed_offsets start (entries): the packs before it hold k*B+1 each
int64_t po_off(const pk_plan* plan, int p, int32_t B)
{
    return (int64_t)plan->packs[p].first_slot * B + p;
}

struct Ws {
    char* base;
    Layout L;
    template <typename T> T* at(size_t off) const { return reinterpret_cast<T*>(base + off); }
};

pk_status check_common(const pk_plan* plan, int32_t B, int64_t nnz, const void* ws, size_t ws_bytes, const char* who,
                       size_t room = ~(size_t)0)
{
    if (!plan) return fail(PK_EINVAL, std::string(who) + ": plan is NULL");
    if (B <= 0) return fail(PK_ESHAPE, std::string(who) + ": B must be positive");
    if (nnz < 0) return fail(PK_ESHAPE, std::string(who) + ": nnz must be non-negative");
    if (nnz > kNnzMax) return fail(PK_EOVERFLOW, std::string(who) + ": nnz must be at most 2^31 - 8192");
    if (plan->opts.max_batch > 0 && B > plan->opts.max_batch) return fail(PK_ESHAPE, std::string(who) + ": B exceeds the plan's max_batch");
    if (plan->opts.max_nnz > 0 && nnz > plan->opts.max_nnz) return fail(PK_ESHAPE, std::string(who) + ": nnz exceeds the plan's max_nnz");
    if ((int64_t)B * plan->out_dim >= ((int64_t)1 << 32)) return fail(PK_EOVERFLOW, std::string(who) + ": B * out_dim must be below 2^32");
    if ((int64_t)B * (int64_t)plan->fields.size() >= ((int64_t)1 << 31)) return fail(PK_EOVERFLOW, std::string(who) + ": n_fields * B must be below 2^31");
    if (!ws) return fail(PK_EINVAL, std::string(who) + ": workspace is NULL");
    if (reinterpret_cast<uintptr_t>(ws) % kAlign) return fail(PK_EWORKSPACE, std::string(who) + ": workspace must be 256-byte aligned");
    if (ws_bytes < make_layout(plan, B, nnz, room).total) return fail(PK_EWORKSPACE, std::string(who) + ": workspace is smaller than pk_workspace_bytes");
    return PK_OK;
}

// The pooling of the packs in `packs` (indices, widest rows first) as one launch's work, from `job`'s sources.
// Runs of up to kRunMax bags per lane group, shorter ones where the launch would have too few wavefronts
// to fill the chip (256 CUs x 16) and where bags hold several IDs: a wavefront takes as long as its longest run,
// and a round of eight positions is full with fewer bags (runs of 8, 4, 2 bags: 1000 fields of 5.5 IDs 222, 209,
// 205 us, 200 fields of 25 IDs 299, 285, 285 us and the step 1568, 1566, 1553).
void fill_pool_job(const pk_plan* plan, const DeviceState* ds, const std::vector<int>& packs, void* const* W, const HotView* hot,
                   int32_t B, int64_t nnz, PoolJob* job)
{
    const int64_t n_bags = (int64_t)B * (int64_t)plan->fields.size();
    int run = kRunMax;
    while (run > 2 && nnz * run >= 16 * n_bags) run /= 2;          // (eight positions or more in the shorter run)
    for (; run > 1; run /= 2) {
        int64_t waves = 0;
        for (int p : packs) {
            const int64_t tile = (int64_t)(64 >> lane_shift(plan->packs[p].dim)) * run;
            waves += (int64_t)plan->packs[p].fields.size() * ((B + tile - 1) / tile);
        }
        if (waves >= 256 * 16) break;
    }
    int64_t items = 0;
    job->n_packs = 0;
    for (int p : packs) {
        const Pack& k = plan->packs[p];
        PoolPack& q = job->pack[job->n_packs++];
        q = PoolPack{};
        q.W = W[p]; q.hv = hot ? hot[p] : HotView{nullptr, nullptr, nullptr}; q.slot_field = ds->slot_field + k.first_slot;
        q.rows = (uint32_t)k.rows; q.po_begin = (uint32_t)po_off(plan, p, B);
        q.D = k.dim; q.sh = lane_shift(k.dim); q.kind = (k.dtype == PK_BF16 ? 1 : 0) | (k.dim < 4 ? 2 : 0);
        const int tile = (64 >> q.sh) * run;
        q.n_fields = (int32_t)k.fields.size(); q.run = run; q.tiles = (B + tile - 1) / tile;
        q.item_begin = (int32_t)items; q.p = p;
        items += (int64_t)q.n_fields * q.tiles;
    }
    job->B = B; job->n_fields = (int32_t)plan->fields.size(); job->fmeta = ds->fmeta; job->n_items = (int32_t)items;
}

template <typename WT>
pk_status hh_swap(DeviceState* ds, hipStream_t stream, const pk_hh_pack& h, int64_t n_hot_old, int64_t n_new, int D,
                  const int32_t* evict_slot, const uint32_t* ins_row, const uint32_t* counts)
{
    // how many rows move is only known on the device; the grids cover the most that can
    const unsigned grid = blocks_for(std::max<int64_t>(n_new, n_hot_old), NT / 64, 4096);
    PK_LAUNCH("pk_hh_evict", pk_hh_evict_kernel<WT>, dim3(grid), dim3(NT), 0, static_cast<WT*>(h.W_cold), h.A_cold,
              static_cast<const WT*>(h.W_hot), h.A_hot, h.hot_row, h.slot_of, evict_slot, counts, D);
    PK_LAUNCH("pk_hh_insert", pk_hh_insert_kernel<WT>, dim3(grid), dim3(NT), 0, static_cast<const WT*>(h.W_cold),
              h.A_cold, static_cast<WT*>(h.W_hot), h.A_hot, h.hot_row, h.slot_of, evict_slot, ins_row, counts, n_hot_old,
              h.hot_rows, D);
    return PK_OK;
}
