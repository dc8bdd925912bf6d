// Executor: turns a plan's executed phases into kernel launches on a HIP
// stream, plus the timing API and the executor options.
//
// An execution is a list of stages (schedule.cpp): phase launches, where the
// steps of one phase with the same source count k (copies are k = 1) run as
// one launch of phase_kernel<dtype, k, aligned, cache mode>, and sliced
// launches of runs of phases (sliced_kernel, or resident_kernel).  Kernels
// read each step as a record holding its range and its resolved buffer
// pointers (StepHead); the records of a buffer set, followed by its n buffer
// pointers, are built on the host and uploaded once, and a small per-plan
// cache keeps them per device, so repeated executes on the same buffers
// launch kernels only.  The tile, sliced and resident tables are uploaded on
// the first execute on a device.  Buffers that are not 16-byte aligned run
// every phase as its phase launches (phase_any_kernel when each is at its
// element's alignment).  A plan that leaves one value in every buffer may
// instead run as one launch of onepass_kernel or onepass_team_kernel, which
// needs its own small tables and the buffer pointers alone.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <tuple>
#include <new>
#include <string>
#include <vector>

#include "exec_state.hpp"
#include "internal.hpp"

namespace arp {

namespace {

std::string hip_msg(const char* what, hipError_t e) {
    return std::string(what) + ": " + hipGetErrorName(e) + " (" +
           hipGetErrorString(e) + ")";
}

}  // namespace

static void free_dev(DevState* d) {
    if (!d) return;
    int cur = -1;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(d->device);
    if (d->tiles) (void)hipFree(d->tiles);
    if (d->cuts) (void)hipFree(d->cuts);
    if (d->sched_off) (void)hipFree(d->sched_off);
    if (d->sched) (void)hipFree(d->sched);
    if (d->stiles) (void)hipFree(d->stiles);
    if (d->runits) (void)hipFree(d->runits);
    if (d->prog) (void)hipFree(d->prog);
    if (d->one_segs) (void)hipFree(d->one_segs);
    if (d->one_prog) (void)hipFree(d->one_prog);
    if (d->one_tiles) (void)hipFree(d->one_tiles);
    for (PtrEntry* c : {d->cache, d->one_cache})
        for (int i = 0; i < kCache; ++i) {
            PtrEntry& e = c[i];
            if (e.done) {
                (void)hipEventSynchronize(e.done);
                (void)hipEventDestroy(e.done);
            }
            if (e.dev) (void)hipFree(e.dev);
            if (e.pinned) (void)hipHostFree(e.pinned);
        }
    if (cur >= 0) (void)hipSetDevice(cur);
    delete d;
}

void exec_release(Plan& p) {
    if (!p.exec) return;
    for (DevState* d : p.exec->dev) free_dev(d);
    delete p.exec;
    p.exec = nullptr;
}

template <class T>
static ar_status upload(T** dst, const std::vector<T>& src, const char* what) {
    if (src.empty()) return AR_OK;
    hipError_t e = hipMalloc(reinterpret_cast<void**>(dst), src.size() * sizeof(T));
    if (e != hipSuccess) {
        *dst = nullptr;
        (void)hipGetLastError();
        return fail(e == hipErrorOutOfMemory ? AR_ERR_OOM : AR_ERR_HIP,
                    hip_msg(what, e));
    }
    e = hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(*dst);
        *dst = nullptr;
        return fail(AR_ERR_HIP, hip_msg(what, e));
    }
    return AR_OK;
}

// The sliced launches' tables of all slices, concatenated (each slice
// indexes them from its *_base offsets).
struct SliceTables {
    std::vector<int64_t> cuts;
    std::vector<int32_t> soff, sched;
    std::vector<int2> tiles;
    std::vector<ResUnit> runits;
    std::vector<uint32_t> prog;
};

static SliceTables slice_tables(const ExecState& ex) {
    SliceTables t;
    for (const SliceDesc& sd : ex.slices) {
        t.cuts.insert(t.cuts.end(), sd.cuts.begin(), sd.cuts.end());
        t.soff.insert(t.soff.end(), sd.sched_off.begin(), sd.sched_off.end());
        t.sched.insert(t.sched.end(), sd.sched.begin(), sd.sched.end());
        t.tiles.insert(t.tiles.end(), sd.tiles.begin(), sd.tiles.end());
        t.runits.insert(t.runits.end(), sd.runits.begin(), sd.runits.end());
        t.prog.insert(t.prog.end(), sd.prog.begin(), sd.prog.end());
    }
    return t;
}

// The plan's state on the current device, with the tables of the route a
// call takes (`one`: the one-pass launch's).
static ar_status device_state(Plan& p, ExecState& ex, bool one, DevState** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(AR_ERR_HIP, hip_msg("hipGetDevice", e));
    if (dev < 0) return fail(AR_ERR_HIP, "no current device");
    if (size_t(dev) >= ex.dev.size()) ex.dev.resize(size_t(dev) + 1, nullptr);
    if (!ex.dev[size_t(dev)]) {
        ex.dev[size_t(dev)] = new DevState();
        ex.dev[size_t(dev)]->device = dev;
    }
    DevState* d = ex.dev[size_t(dev)];
    ar_status s = AR_OK;
    if (one && !d->one) {
        if (!d->one_segs) s = upload(&d->one_segs, ex.one.segs, "one-pass segments");
        if (s == AR_OK && !d->one_prog) s = upload(&d->one_prog, ex.one.prog, "one-pass leaves");
        if (s == AR_OK && !d->one_tiles) s = upload(&d->one_tiles, ex.one.tiles, "one-pass tiles");
        d->one = s == AR_OK;
    } else if (!one && !d->staged) {
        if (!d->tiles) s = upload(&d->tiles, ex.htiles, "tile table");
        if (s == AR_OK && !ex.slices.empty()) {
            const SliceTables t = slice_tables(ex);
            if (!d->cuts) s = upload(&d->cuts, t.cuts, "segment table");
            if (s == AR_OK && !d->sched_off) s = upload(&d->sched_off, t.soff, "schedule offsets");
            if (s == AR_OK && !d->sched) s = upload(&d->sched, t.sched, "schedule");
            if (s == AR_OK && !d->stiles) s = upload(&d->stiles, t.tiles, "slice tiles");
            if (s == AR_OK && !d->runits) s = upload(&d->runits, t.runits, "resident units");
            if (s == AR_OK && !d->prog) s = upload(&d->prog, t.prog, "resident programs");
        }
        d->staged = s == AR_OK;
    }
    if (s != AR_OK) return s;
    *out = d;
    (void)p;
    return AR_OK;
}

// Host-side checks of the buffer set: non-NULL and pairwise disjoint.
static ar_status check_buffers(const Plan& p, const std::vector<void*>& bufs) {
    const uint64_t bytes = uint64_t(p.N) * uint64_t(p.esize);
    std::vector<std::pair<uint64_t, int32_t>> a;
    a.reserve(bufs.size());
    for (size_t i = 0; i < bufs.size(); ++i) {
        if (!bufs[i])
            return fail(AR_ERR_INVALID_ARG, "buffer " + std::to_string(i) + " is NULL");
        a.emplace_back(reinterpret_cast<uint64_t>(bufs[i]), int32_t(i));
    }
    std::sort(a.begin(), a.end());
    for (size_t i = 1; i < a.size(); ++i)
        if (a[i].first < a[i - 1].first + bytes)
            return fail(AR_ERR_INVALID_ARG,
                        "buffers " + std::to_string(a[i - 1].second) + " and " +
                            std::to_string(a[i].second) + " overlap");
    return AR_OK;
}

// What every buffer is aligned to: 16 bytes, its element (16-byte accesses at
// element alignment), or less (element-wise).
enum Align { ALIGN_NONE, ALIGN_ELEM, ALIGN_16 };
static Align buffers_align(void* const* bufs, int32_t n, int32_t esize) {
    uint64_t any = 0;
    for (int32_t i = 0; i < n; ++i) any |= reinterpret_cast<uint64_t>(bufs[i]);
    return !(any & 15) ? ALIGN_16 : !(any & uint64_t(esize - 1)) ? ALIGN_ELEM : ALIGN_NONE;
}

// Does a call on these buffers run the one-pass launch?  (Its form is built
// here when only unaligned buffers take it.)
static bool takes_one(const Plan& p, ExecState& ex, void* const* bufs) {
    if (!ex.one_aligned && !ex.one_unaligned) return false;
    const Align a = buffers_align(bufs, p.n, p.esize);
    if (a == ALIGN_16) return ex.one_aligned;
    if (!ex.one_unaligned || a != ALIGN_ELEM) return false;
    build_onepass(p, ex, ex.one);
    return ex.one.ok;
}

// The step records of buffer set bufs[0..n) (see StepHead) followed by the n
// buffer pointers, written to w[0 .. rec_words + n).
static void fill_records(const ExecState& ex, void* const* bufs, int32_t n, uint64_t* w) {
    std::memset(w, 0, size_t(ex.rec_words + n) * sizeof(uint64_t));
    for (size_t i = 0; i < ex.hsteps.size(); ++i) {
        const DevStep& st = ex.hsteps[i];
        uint64_t* r = w + ex.rec_of[i];
        StepHead h{st.begin, st.end, st.k, st.ndst, st.nfree, 0};
        std::memcpy(r, &h, sizeof(h));
        for (int32_t j = 0; j < st.k; ++j)
            r[kRecHead + j] = reinterpret_cast<uint64_t>(bufs[size_t(ex.hidx[size_t(st.src_off + j)])]);
        for (int32_t j = 0; j < st.ndst; ++j)
            r[kRecHead + st.k + j] =
                reinterpret_cast<uint64_t>(bufs[size_t(ex.hidx[size_t(st.dst_off + j)])]);
    }
    for (int32_t i = 0; i < n; ++i) w[ex.rec_words + i] = reinterpret_cast<uint64_t>(bufs[i]);
}

// The step records for buffer set `bufs` on this device (see StepHead),
// followed by the n buffer pointers (`one`: the pointers alone): from the
// per-plan cache, or built on the host and uploaded on `stream`.
static ar_status step_records(const Plan& p, const ExecState& ex, DevState& d,
                              const std::vector<void*>& bufs, bool one,
                              hipStream_t stream, PtrEntry** out) {
    PtrEntry* const cache = one ? d.one_cache : d.cache;
    ++d.clock;
    for (int i = 0; i < kCache; ++i)
        if (cache[i].valid && cache[i].key == bufs) {
            cache[i].stamp = d.clock;
            *out = &cache[i];
            return AR_OK;
        }
    ar_status s = check_buffers(p, bufs);
    if (s != AR_OK) return s;
    PtrEntry* v = &cache[0];
    for (int i = 0; i < kCache; ++i) {
        if (!cache[i].valid) { v = &cache[i]; break; }
        if (cache[i].stamp < v->stamp) v = &cache[i];
    }
    const size_t nb = size_t((one ? 0 : ex.rec_words) + p.n) * sizeof(uint64_t);
    hipError_t e = hipSuccess;
    if (!v->dev) {
        e = hipMalloc(reinterpret_cast<void**>(&v->dev), nb);
        if (e != hipSuccess) {
            v->dev = nullptr;
            (void)hipGetLastError();
            return fail(e == hipErrorOutOfMemory ? AR_ERR_OOM : AR_ERR_HIP, hip_msg("step records", e));
        }
        e = hipHostMalloc(reinterpret_cast<void**>(&v->pinned), nb, hipHostMallocDefault);
        if (e != hipSuccess) {
            v->pinned = nullptr;
            (void)hipGetLastError();
            return fail(AR_ERR_OOM, hip_msg("step record staging", e));
        }
        e = hipEventCreateWithFlags(&v->done, hipEventDisableTiming);
        if (e != hipSuccess) {
            v->done = nullptr;
            return fail(AR_ERR_HIP, hip_msg("hipEventCreate", e));
        }
    } else {
        // the previous upload from the staging buffer must have finished
        e = hipEventSynchronize(v->done);
        if (e != hipSuccess) return fail(AR_ERR_HIP, hip_msg("hipEventSynchronize", e));
    }
    v->valid = false;
    if (one) std::memcpy(v->pinned, bufs.data(), nb);
    else fill_records(ex, bufs.data(), p.n, v->pinned);
    e = hipMemcpyAsync(v->dev, v->pinned, nb, hipMemcpyHostToDevice, stream);
    if (e != hipSuccess) return fail(AR_ERR_HIP, hip_msg("step record upload", e));
    e = hipEventRecord(v->done, stream);
    if (e != hipSuccess) return fail(AR_ERR_HIP, hip_msg("hipEventRecord", e));
    v->key = bufs;
    v->valid = true;
    v->stamp = d.clock;
    v->align = buffers_align(bufs.data(), p.n, p.esize);
    *out = v;
    return AR_OK;
}

// align: the buffers' (Align).
template <int DT, int K>
static void launch_dk(int align, int cm, int64_t blocks, hipStream_t st,
                      const uint64_t* recs, int64_t stride, const int2* tiles,
                      int64_t nunits, int64_t tps, int64_t te, int rtg,
                      int dsplit, int wide, int narrow) {
    const dim3 block(64 * kcfg(K).WPB);
    const bool vecok = align == ALIGN_16;
    if constexpr (K == 2) {
        if (wide && vecok && cm == 3 && dsplit == 1) {  // see kWideBytes
            hipLaunchKernelGGL((phase_kernel<DT, 2, true, 3, kWideU>),
                               dim3(static_cast<uint32_t>(blocks)), block, 0, st, recs, stride,
                               tiles, nunits, tps, te, rtg);
            return;
        }
    }
    if constexpr (K == 8 && DT != DT_BF16) {
        if (wide && vecok && (cm & 1) && dsplit == 1) {  // see kWideBytes
            if (cm & 2)
                hipLaunchKernelGGL((phase_kernel<DT, 8, true, 3, kWideU8>),
                                   dim3(static_cast<uint32_t>(blocks)), block, 0, st, recs,
                                   stride, tiles, nunits, tps, te, rtg);
            else
                hipLaunchKernelGGL((phase_kernel<DT, 8, true, 1, kWideU8>),
                                   dim3(static_cast<uint32_t>(blocks)), block, 0, st, recs,
                                   stride, tiles, nunits, tps, te, rtg);
            return;
        }
    }
    if (dsplit > 1 && vecok) {  // a workgroup per table entry
        // the waves of a workgroup all read the tile's sources: cached loads
        // (with nontemporal ones each wave fetched them from memory again)
        const int64_t ntiles = nunits / dsplit;
        const dim3 grid(static_cast<uint32_t>(ntiles)), sblock(64 * kSplitWaves);
        if (cm & 2)
            hipLaunchKernelGGL((split_kernel<DT, K, 2>), grid, sblock, 0, st, recs, stride, tiles,
                               ntiles, te, rtg);
        else
            hipLaunchKernelGGL((split_kernel<DT, K, 0>), grid, sblock, 0, st, recs, stride, tiles,
                               ntiles, te, rtg);
        return;
    }
    if (dsplit > 1) {  // unaligned buffers: one wave per table entry
        nunits /= dsplit;
        blocks = (nunits + kcfg(K).WPB - 1) / kcfg(K).WPB;
    }
    const dim3 grid(static_cast<uint32_t>(blocks));
    constexpr int kNarrowU = K == 0 ? kNarrowU0 : K == 1 ? kNarrowU1 : 0;  // see kNarrowMinSrc
#define AR_LAUNCH(V, C)                                                                \
    hipLaunchKernelGGL((phase_kernel<DT, K, V, C>), grid, block, 0, st, recs, stride, \
                       tiles, nunits, tps, te, rtg)
    if (align == ALIGN_ELEM)
        hipLaunchKernelGGL((phase_any_kernel<DT, K>), grid, block, 0, st, recs, stride, tiles,
                           nunits, tps, te);
    else if (!vecok) AR_LAUNCH(false, 0);
    else if (cm == 0 && narrow)
        hipLaunchKernelGGL((phase_kernel<DT, K, true, 0, kNarrowU>), grid, block, 0, st, recs,
                           stride, tiles, nunits, tps, te, rtg);
    else if (cm == 0) AR_LAUNCH(true, 0);
    else if (cm == 1) AR_LAUNCH(true, 1);
    else if (cm == 2) AR_LAUNCH(true, 2);
    else AR_LAUNCH(true, 3);
#undef AR_LAUNCH
}

template <int DT>
static void launch_d(int K, int align, int cm, int64_t blocks, hipStream_t st,
                     const uint64_t* recs, int64_t stride, const int2* tiles,
                     int64_t nunits, int64_t tps, int64_t te, int rtg,
                     int dsplit, int wide, int narrow) {
    switch (K) {
        case 1: launch_dk<DT, 1>(align, cm, blocks, st, recs, stride, tiles, nunits, tps, te, rtg, dsplit, wide, narrow); break;
        case 2: launch_dk<DT, 2>(align, cm, blocks, st, recs, stride, tiles, nunits, tps, te, rtg, dsplit, wide, narrow); break;
        case 3: launch_dk<DT, 3>(align, cm, blocks, st, recs, stride, tiles, nunits, tps, te, rtg, dsplit, wide, narrow); break;
        case 4: launch_dk<DT, 4>(align, cm, blocks, st, recs, stride, tiles, nunits, tps, te, rtg, dsplit, wide, narrow); break;
        case 8: launch_dk<DT, 8>(align, cm, blocks, st, recs, stride, tiles, nunits, tps, te, rtg, dsplit, wide, narrow); break;
        case 16: launch_dk<DT, 16>(align, cm, blocks, st, recs, stride, tiles, nunits, tps, te, rtg, dsplit, wide, narrow); break;
        default: launch_dk<DT, 0>(align, cm, blocks, st, recs, stride, tiles, nunits, tps, te, rtg, dsplit, wide, narrow); break;
    }
}

}  // namespace arp

struct ar_timer {
    int64_t cap = 0;
    int64_t count = 0;
    std::vector<hipEvent_t> ev;  // 2 per record, created lazily
    std::vector<int32_t> launch;
};

using namespace arp;

// Where one execution's device-side tables and step records are: the
// plan's own device state, or the no-allocation entry point's scratch.
struct DevView {
    const int2* tiles;
    const int64_t* cuts;
    const int32_t* sched_off;
    const int32_t* sched;
    const int2* stiles;
    const ResUnit* runits;
    const uint32_t* prog;
    const uint64_t* recs;  // step records, then the n buffer pointers
    int align;             // the buffers' (Align)
    // the one-pass launch, when the call takes it: its tables, the pointers
    bool one = false;
    const OneSeg* one_segs = nullptr;
    const uint32_t* one_prog = nullptr;
    const int2* one_tiles = nullptr;
    const uint64_t* ptrs = nullptr;
};

template <int DT, int LB, int U, int B, int W>
static void launch_one(const Plan& p, const OnePlan& one, const DevView& v, hipStream_t stream) {
    const int64_t blocks = (one.nunits + W - 1) / W;
    const bool many = U == 1 && W == 1 && one.many >= (v.align == ALIGN_16 ? 1 : 2);
    const uint32_t per_xcd = many ? 0u : static_cast<uint32_t>((blocks + 7) / 8);
    const dim3 grid(many ? static_cast<uint32_t>(blocks) : per_xcd * 8), block(64 * W);
    const size_t lds = std::max(size_t(one.depth) * U * 64 * W * sizeof(typename OneVec<DT, LB>::Acc),
                                many ? size_t(one_lds(p.n)) : size_t(0));
    const int32_t amask = v.align == ALIGN_16 ? LB / p.esize - 1 : 0;
#define AR_ONE(CM)                                                                            \
    hipLaunchKernelGGL((onepass_kernel<DT, LB, U, B, W, CM>), grid, block, lds, stream, v.ptrs,   \
                       p.n, v.one_prog, v.one_segs, int32_t(one.segs.size()), v.one_tiles,    \
                       uint32_t(one.nunits), uint32_t(one.tiles_per_seg), per_xcd, p.N, amask)
    if (one.cm == 3) AR_ONE(3);
    else AR_ONE(0);
#undef AR_ONE
}

template <int DT, int W, int LPW>
static void launch_team(const Plan& p, const OnePlan& one, const DevView& v, hipStream_t stream) {
    const uint32_t per_xcd = static_cast<uint32_t>((one.nunits + 7) / 8);
    const size_t lds = size_t(2 * W * LPW * 64 + 64) * 4 +
                       size_t(one.depth) * 64 * sizeof(typename OneVec<DT, 4>::Acc);
    hipLaunchKernelGGL((onepass_team_kernel<DT, W, LPW>), dim3(per_xcd * 8), dim3(64 * W), lds, stream,
                       v.ptrs, p.n, v.one_prog, v.one_segs, int32_t(one.segs.size()), v.one_tiles,
                       uint32_t(one.nunits), uint32_t(one.tiles_per_seg), per_xcd, p.N,
                       v.align == ALIGN_16 ? 4 / p.esize - 1 : 0);
}

template <int DT>
static void launch_one_d(const Plan& p, const OnePlan& one, const DevView& v, hipStream_t stream) {
    switch (one.conf.kind) {
        case ONE_LB4: launch_one<DT, 4, 1, 32, 4>(p, one, v, stream); break;
        case ONE_U4: launch_one<DT, 16, 4, 4, 1>(p, one, v, stream); break;
        case ONE_U8: launch_one<DT, 16, 8, 2, 1>(p, one, v, stream); break;
        case ONE_U16: launch_one<DT, 16, 16, 1, 1>(p, one, v, stream); break;
        case ONE_TEAM4: launch_team<DT, 4, 16>(p, one, v, stream); break;
        case ONE_TEAM16: launch_team<DT, 16, 8>(p, one, v, stream); break;
        case ONE_U1B4: launch_one<DT, 16, 1, 4, 1>(p, one, v, stream); break;
        case ONE_U1B8: launch_one<DT, 16, 1, 8, 1>(p, one, v, stream); break;
        default: launch_one<DT, 16, 1, 16, 1>(p, one, v, stream); break;
    }
}

// Enqueue the launches of one execution on `stream`.
static ar_status launch_all(ar_plan* plan, const ExecState* ex, const DevView& v,
                            hipStream_t stream, ar_timer* timer) {
    const DevView* d = &v;
    ar_status s = AR_OK;
    {
        // sliced launches need 16-byte aligned buffers; otherwise every
        // phase runs as its phase launches
        const bool staged = v.align == ALIGN_16;
        const int64_t nlaunch = v.one ? 1
                                : staged ? int64_t(ex->run_stages.size()) : int64_t(ex->launches.size());
        if (timer && timer->count + nlaunch > timer->cap)
            return fail(AR_ERR_INVALID_ARG, "timer is full");
        auto mark = [&](int j) -> ar_status {  // event j (0 begin, 1 end) of this record
            if (!timer) return AR_OK;
            hipEvent_t& ev = timer->ev[size_t(2 * timer->count + j)];
            if (!ev) {
                hipError_t he = hipEventCreate(&ev);
                if (he != hipSuccess) {
                    ev = nullptr;
                    return fail(AR_ERR_HIP, hip_msg("hipEventCreate", he));
                }
            }
            hipError_t he = hipEventRecord(ev, stream);
            if (he != hipSuccess) return fail(AR_ERR_HIP, hip_msg("hipEventRecord", he));
            return AR_OK;
        };
        for (int64_t li = 0; li < nlaunch; ++li) {
            s = mark(0);
            if (s != AR_OK) return s;
            const Stage stg = v.one    ? Stage{-1, -1}
                              : staged ? ex->run_stages[size_t(li)] : Stage{-1, int32_t(li)};
            if (v.one) {
                switch (plan->dtype) {
                    case AR_F32: launch_one_d<DT_F32>(*plan, ex->one, v, stream); break;
                    case AR_I32: launch_one_d<DT_I32>(*plan, ex->one, v, stream); break;
                    default: launch_one_d<DT_BF16>(*plan, ex->one, v, stream); break;
                }
            } else if (stg.slice >= 0 && ex->slices[size_t(stg.slice)].streamed) {
                const SliceDesc& sd = ex->slices[size_t(stg.slice)];
                if (sd.res_waves != 4) return fail(AR_ERR_INTERNAL, "streamed launch shape");
                const dim3 grid(static_cast<uint32_t>(sd.nunits)), block(256);
                // the slots, the n buffer pointers, the longest unit program
                const size_t lds = size_t(sd.slots) * 1024 + size_t(plan->n) * 8 + size_t(sd.max_nw) * 4;
                const bool nt = sd.res_bytes > 2 * kKeepBytes;
#define AR_STREAM_K(DT, W, NT)                                                                \
    hipLaunchKernelGGL((stream_kernel<DT, W, NT>), grid, block, lds, stream,                    \
                       v.recs + ex->rec_words, plan->n, sd.slots,                              \
                       d->runits + sd.runit_base, d->prog + sd.prog_base, sd.nunits)
#define AR_STREAM(DT)                                                                         \
    if (nt) AR_STREAM_K(DT, 4, true);                                                         \
    else AR_STREAM_K(DT, 4, false)
                switch (plan->dtype) {
                    case AR_F32: AR_STREAM(DT_F32); break;
                    case AR_I32: AR_STREAM(DT_I32); break;
                    default: AR_STREAM(DT_BF16); break;
                }
#undef AR_STREAM
#undef AR_STREAM_K
            } else if (stg.slice >= 0 && ex->slices[size_t(stg.slice)].resident) {
                const SliceDesc& sd = ex->slices[size_t(stg.slice)];
                const dim3 grid(static_cast<uint32_t>(sd.nunits)), block(64 * sd.res_waves);
                const size_t lds = size_t(plan->n) * 1024;
#define AR_RESIDENT(DT, W, NT)                                                                \
    hipLaunchKernelGGL((resident_kernel<DT, W, NT>), grid, block, lds, stream,                \
                       v.recs + ex->rec_words, plan->n, d->runits + sd.runit_base,           \
                       d->prog + sd.prog_base, sd.nunits)
                // runs moving more than the last-level cache holds stream
                // their rows past it
                const bool nt = sd.res_bytes > 2 * kKeepBytes;
#define AR_RESIDENT_W(DT)                                                                     \
    if (sd.res_waves == 4) {                                                                  \
        if (nt) AR_RESIDENT(DT, 4, true); else AR_RESIDENT(DT, 4, false);                     \
    } else {                                                                                  \
        if (nt) AR_RESIDENT(DT, 1, true); else AR_RESIDENT(DT, 1, false);                     \
    }
                switch (plan->dtype) {
                    case AR_F32: AR_RESIDENT_W(DT_F32); break;
                    case AR_I32: AR_RESIDENT_W(DT_I32); break;
                    default: AR_RESIDENT_W(DT_BF16); break;
                }
#undef AR_RESIDENT_W
#undef AR_RESIDENT
            } else if (stg.slice >= 0) {
                const SliceDesc& sd = ex->slices[size_t(stg.slice)];
                const dim3 grid(static_cast<uint32_t>((sd.nunits + kSliceWPB - 1) / kSliceWPB));
                const dim3 block(64 * kSliceWPB);
#define AR_SLICED(DT)                                                                   \
    hipLaunchKernelGGL((sliced_kernel<DT>), grid, block, 0, stream, v.recs,             \
                       d->sched_off + sd.soff_base, d->sched + sd.sched_base,           \
                       d->cuts + sd.cuts_base, d->stiles + sd.tiles_base, sd.nunits,    \
                       sd.nphases, sd.nseg, sd.tile_elems)
                switch (plan->dtype) {
                    case AR_F32: AR_SLICED(DT_F32); break;
                    case AR_I32: AR_SLICED(DT_I32); break;
                    default: AR_SLICED(DT_BF16); break;
                }
#undef AR_SLICED
            } else {
                const LaunchDesc& L = ex->launches[size_t(stg.launch)];
                const int64_t blocks = (L.nunits + L.wpb - 1) / L.wpb;
                const uint64_t* recs = v.recs + L.rec_off;
                const int2* tiles = L.tile_off >= 0 ? d->tiles + L.tile_off : nullptr;
                switch (plan->dtype) {
                    case AR_F32:
                        launch_d<DT_F32>(L.kern_k, v.align, L.cm, blocks, stream, recs,
                                         L.rec_stride, tiles, L.nunits, L.tiles_per_step,
                                         L.tile_elems, L.rt_group, L.dsplit, L.wide,
                                         L.narrow);
                        break;
                    case AR_I32:
                        launch_d<DT_I32>(L.kern_k, v.align, L.cm, blocks, stream, recs,
                                         L.rec_stride, tiles, L.nunits, L.tiles_per_step,
                                         L.tile_elems, L.rt_group, L.dsplit, L.wide,
                                         L.narrow);
                        break;
                    default:
                        launch_d<DT_BF16>(L.kern_k, v.align, L.cm, blocks, stream, recs,
                                          L.rec_stride, tiles, L.nunits, L.tiles_per_step,
                                          L.tile_elems, L.rt_group, L.dsplit, L.wide,
                                          L.narrow);
                        break;
                }
            }
            hipError_t he = hipGetLastError();
            if (he != hipSuccess) return fail(AR_ERR_HIP, hip_msg("kernel launch", he));
            s = mark(1);
            if (s != AR_OK) return s;
            if (timer) timer->launch[size_t(timer->count++)] = int32_t(li);
        }
    }
    return AR_OK;
}

static ar_status run(ar_plan* plan, const std::vector<void*>& bufs,
                     hipStream_t stream, ar_timer* timer) {
    try {
        if (plan->N == 0 || plan->num_phases() == 0) return AR_OK;
        ExecState* ex = exec_state(*plan);
        if (ex->launches.empty()) return AR_OK;
        const bool one = takes_one(*plan, *ex, bufs.data());
        DevState* d = nullptr;
        ar_status s = device_state(*plan, *ex, one, &d);
        if (s != AR_OK) return s;
        PtrEntry* pe = nullptr;
        s = step_records(*plan, *ex, *d, bufs, one, stream, &pe);
        if (s != AR_OK) return s;
        DevView v{d->tiles, d->cuts, d->sched_off, d->sched, d->stiles,
                  d->runits, d->prog, pe->dev, pe->align};
        if (one) {
            v.one = true;
            v.one_segs = d->one_segs;
            v.one_prog = d->one_prog;
            v.one_tiles = d->one_tiles;
            v.ptrs = pe->dev;
        }
        return launch_all(plan, ex, v, stream, timer);
    } catch (const std::bad_alloc&) {
        return fail(AR_ERR_OOM, "host allocation failed");
    } catch (const std::exception& e) {
        return fail(AR_ERR_INTERNAL, e.what());
    }
}

// ------------------------------------------- execution without allocation
//
// ar_plan_execute_noalloc keeps an execution's device-side tables and step
// records in `scratch`, a fixed array of this library on every device (no
// device allocation at any call).  Host code never uses the array's name
// as an address: on a device's first call the device address comes from
// hipGetSymbolAddress with that device current, and is kept per device.
// Calls on one device share the array.  An executor state's image has a place
// of its own from its first call on (a graph that captured the launches reads
// it there), one after the other and from the start again when the end is
// reached.  The host remembers which images the array holds, with which buffer
// sets, and copies one only when it is not there (three plans in turn, Ring
// n = 4 over 2^16 int32: 9.9 us a call with a copy of 13 KiB each, 6.4
// without).

static __device__ __align__(256) uint8_t scratch[AR_NOALLOC_MAX_BYTES];

namespace {

// An image that `scratch` holds: an executor state's tables (of one route)
// with the records of a buffer set, and where.
struct ScratchImage {
    uint64_t serial = 0;
    bool one = false;             // the one-pass launch's tables
    std::vector<void*> bufs;
    int64_t off = 0, size = 0;
};
struct ScratchDev {
    uint8_t* ptr = nullptr;       // device address of `scratch` on this device
    uint64_t last = 0;            // serial of the last call's executor state
    std::vector<ScratchImage> held;
};
// Images kept at most: a program's plans in turn; each call looks through them.
constexpr size_t kScratchImages = 32;
std::mutex g_scratch_mu;
std::vector<ScratchDev> g_scratch;  // by device ordinal
int64_t g_scratch_next = 0;         // where the next image is placed

constexpr int64_t kImgAlign = 256;

// Is `st` being captured into a graph?  (The null stream cannot be.)
bool capturing(hipStream_t st) {
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    return st && hipStreamIsCapturing(st, &s) == hipSuccess && s != hipStreamCaptureStatusNone;
}

int64_t img_align(int64_t b) { return (b + kImgAlign - 1) / kImgAlign * kImgAlign; }

}  // namespace

// Bytes of the image of `ex`: its tables and the records of one buffer set.
// The limit holds for this size, whichever launches the call runs.
static int64_t image_bytes(const Plan& p, const ExecState& ex) {
    size_t cuts = 0, soff = 0, sched = 0, tiles = 0, runits = 0, prog = 0;
    for (const SliceDesc& sd : ex.slices) {
        cuts += sd.cuts.size();
        soff += sd.sched_off.size();
        sched += sd.sched.size();
        tiles += sd.tiles.size();
        runits += sd.runits.size();
        prog += sd.prog.size();
    }
    int64_t at = 0;
    for (size_t b : {ex.htiles.size() * sizeof(int2), cuts * sizeof(int64_t), soff * sizeof(int32_t),
                     sched * sizeof(int32_t), tiles * sizeof(int2), runits * sizeof(ResUnit),
                     prog * sizeof(uint32_t), size_t(ex.rec_words + p.n) * sizeof(uint64_t)})
        at = img_align(at + int64_t(b));
    return at;
}

// Lay out the tables of `ex` and room for the records of one buffer set in
// ex->img.
static void build_image(const Plan& p, ExecState& ex) {
    const SliceTables t = slice_tables(ex);
    const int64_t sizes[8] = {
        int64_t(ex.htiles.size() * sizeof(int2)), int64_t(t.cuts.size() * sizeof(int64_t)),
        int64_t(t.soff.size() * sizeof(int32_t)), int64_t(t.sched.size() * sizeof(int32_t)),
        int64_t(t.tiles.size() * sizeof(int2)),   int64_t(t.runits.size() * sizeof(ResUnit)),
        int64_t(t.prog.size() * sizeof(uint32_t)),
        (ex.rec_words + p.n) * int64_t(sizeof(uint64_t))};
    int64_t at = 0;
    for (int i = 0; i < 8; ++i) {
        ex.img_off[i] = at;
        at = img_align(at + sizes[i]);
    }
    ex.img.assign(size_t(at / 8), 0);
    char* b = reinterpret_cast<char*>(ex.img.data());
    const void* src[7] = {ex.htiles.data(), t.cuts.data(), t.soff.data(), t.sched.data(),
                          t.tiles.data(), t.runits.data(), t.prog.data()};
    for (int i = 0; i < 7; ++i)
        if (sizes[i]) std::memcpy(b + ex.img_off[i], src[i], size_t(sizes[i]));
}

// The same for the one-pass launch: segments, leaves, tiles, then room for
// the n buffer pointers; empty when it exceeds the array.
static void build_one_image(const Plan& p, ExecState& ex) {
    const OnePlan& o = ex.one;
    const int64_t sizes[4] = {
        int64_t(o.segs.size() * sizeof(OneSeg)), int64_t(o.prog.size() * sizeof(uint32_t)),
        int64_t(o.tiles.size() * sizeof(int2)), int64_t(p.n) * int64_t(sizeof(uint64_t))};
    int64_t at = 0;
    for (int i = 0; i < 4; ++i) {
        ex.one_img_off[i] = at;
        at = img_align(at + sizes[i]);
    }
    if (at > int64_t(AR_NOALLOC_MAX_BYTES)) return;
    ex.one_img.assign(size_t(at / 8), 0);
    char* b = reinterpret_cast<char*>(ex.one_img.data());
    const void* src[3] = {o.segs.data(), o.prog.data(), o.tiles.data()};
    for (int i = 0; i < 3; ++i)
        if (sizes[i]) std::memcpy(b + ex.one_img_off[i], src[i], size_t(sizes[i]));
}

AR_EXPORT ar_status ar_plan_execute_noalloc(ar_plan* plan, void* const* bufs, void* stream) {
    clear_error();
    if (!plan) return fail(AR_ERR_INVALID_ARG, "plan is NULL");
    if (!bufs) return fail(AR_ERR_INVALID_ARG, "bufs is NULL");
    try {
        if (plan->N == 0 || plan->num_phases() == 0) return AR_OK;
        ExecState* ex = exec_state(*plan);
        if (ex->launches.empty()) return AR_OK;
        for (int32_t i = 0; i < plan->n; ++i)  // before anything reads their alignment
            if (!bufs[i])
                return fail(AR_ERR_INVALID_ARG, "buffer " + std::to_string(i) + " is NULL");
        bool one = takes_one(*plan, *ex, bufs);
        int dev = -1;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return fail(AR_ERR_HIP, hip_msg("hipGetDevice", e));
        if (dev < 0) return fail(AR_ERR_HIP, "no current device");
        const hipStream_t st = static_cast<hipStream_t>(stream);
        uint8_t* base = nullptr;
        {
            std::lock_guard<std::mutex> lock(g_scratch_mu);
            if (size_t(dev) >= g_scratch.size()) g_scratch.resize(size_t(dev) + 1);
            ScratchDev& sd = g_scratch[size_t(dev)];
            ScratchImage* im = nullptr;  // its tables, whichever the records
            for (ScratchImage& h : sd.held)
                if (h.serial == ex->serial && h.one == one) im = &h;
            // Within a capture only what the last call used counts as there: other
            // images may be replaced before the replays, which then need their
            // own copy.
            const bool last = sd.last == ex->serial;
            if (im && std::equal(im->bufs.begin(), im->bufs.end(), bufs, bufs + plan->n) &&
                (last || !capturing(st))) {
                base = sd.ptr + im->off;
            } else {
                const std::vector<void*> set(bufs, bufs + plan->n);
                ar_status s = check_buffers(*plan, set);
                if (s != AR_OK) return s;
                if (ex->img.empty() && ex->one_img.empty()) {
                    const int64_t need = image_bytes(*plan, *ex);
                    if (need > int64_t(AR_NOALLOC_MAX_BYTES))
                        return fail(AR_ERR_UNSUPPORTED,
                                    "the plan's tables and step records take " +
                                        std::to_string(need) +
                                        " bytes; ar_plan_execute_noalloc holds at most " +
                                        std::to_string(int64_t(AR_NOALLOC_MAX_BYTES)));
                }
                if (one && ex->one_img.empty()) {
                    build_one_image(*plan, *ex);
                    one = !ex->one_img.empty();
                }
                if (!one && ex->img.empty()) build_image(*plan, *ex);
                if (!sd.ptr) {
                    void* ptr = nullptr;
                    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
                    if (e != hipSuccess || !ptr)
                        return fail(AR_ERR_HIP, hip_msg("hipGetSymbolAddress(scratch)", e));
                    sd.ptr = static_cast<uint8_t*>(ptr);
                }
                std::vector<uint64_t>& img = one ? ex->one_img : ex->img;
                const int64_t rec = one ? ex->one_img_off[3] : ex->img_off[7];
                const int64_t size = int64_t(img.size()) * 8;
                int64_t& off = ex->scratch_off[one ? 1 : 0];
                if (off < 0) {
                    if (g_scratch_next + size > int64_t(AR_NOALLOC_MAX_BYTES)) g_scratch_next = 0;
                    off = g_scratch_next;
                    g_scratch_next = img_align(off + size);
                }
                im = nullptr;  // (the route may have changed)
                for (ScratchImage& h : sd.held)
                    if (h.serial == ex->serial && h.one == one) im = &h;
                const bool cap = capturing(st);
                const int64_t from = im && !cap ? rec : 0;
                // what was there is gone (unknown until the copy is enqueued)
                sd.held.erase(std::remove_if(sd.held.begin(), sd.held.end(),
                                             [&](const ScratchImage& h) {
                                                 return h.off < off + size && off < h.off + h.size;
                                             }),
                              sd.held.end());
                if (sd.held.size() >= kScratchImages) sd.held.erase(sd.held.begin());
                uint64_t* const r = img.data() + rec / int64_t(sizeof(uint64_t));
                if (one) std::memcpy(r, bufs, size_t(plan->n) * sizeof(uint64_t));
                else fill_records(*ex, bufs, plan->n, r);
                e = hipMemcpyAsync(sd.ptr + off + from, reinterpret_cast<const char*>(img.data()) + from,
                                   size_t(size - from), hipMemcpyHostToDevice, st);
                if (e != hipSuccess) return fail(AR_ERR_HIP, hip_msg("scratch upload", e));
                // (a captured copy has not run: the next call makes its own)
                if (!cap) sd.held.push_back({ex->serial, one, set, off, size});
                base = sd.ptr + off;
            }
            sd.last = ex->serial;
        }
        if (one) {
            DevView v{};
            v.align = buffers_align(bufs, plan->n, plan->esize);
            v.one = true;
            v.one_segs = reinterpret_cast<const OneSeg*>(base + ex->one_img_off[0]);
            v.one_prog = reinterpret_cast<const uint32_t*>(base + ex->one_img_off[1]);
            if (!ex->one.tiles.empty())
                v.one_tiles = reinterpret_cast<const int2*>(base + ex->one_img_off[2]);
            v.ptrs = reinterpret_cast<const uint64_t*>(base + ex->one_img_off[3]);
            return launch_all(plan, ex, v, st, nullptr);
        }
        auto at = [&](int i) { return base + ex->img_off[i]; };
        const DevView v{reinterpret_cast<const int2*>(at(0)), reinterpret_cast<const int64_t*>(at(1)),
                        reinterpret_cast<const int32_t*>(at(2)), reinterpret_cast<const int32_t*>(at(3)),
                        reinterpret_cast<const int2*>(at(4)), reinterpret_cast<const ResUnit*>(at(5)),
                        reinterpret_cast<const uint32_t*>(at(6)), reinterpret_cast<const uint64_t*>(at(7)),
                        buffers_align(bufs, plan->n, plan->esize)};
        return launch_all(plan, ex, v, st, nullptr);
    } catch (const std::bad_alloc&) {
        return fail(AR_ERR_OOM, "host allocation failed");
    } catch (const std::exception& e) {
        return fail(AR_ERR_INTERNAL, e.what());
    }
}

AR_EXPORT ar_status ar_plan_execute(ar_plan* plan, void* const* bufs, void* stream) {
    clear_error();
    if (!plan) return fail(AR_ERR_INVALID_ARG, "plan is NULL");
    if (!bufs) return fail(AR_ERR_INVALID_ARG, "bufs is NULL");
    return run(plan, std::vector<void*>(bufs, bufs + plan->n),
               static_cast<hipStream_t>(stream), nullptr);
}

AR_EXPORT ar_status ar_plan_execute_timed(ar_plan* plan, void* const* bufs, void* stream,
                                          ar_timer* timer) {
    clear_error();
    if (!plan) return fail(AR_ERR_INVALID_ARG, "plan is NULL");
    if (!bufs) return fail(AR_ERR_INVALID_ARG, "bufs is NULL");
    if (!timer) return fail(AR_ERR_INVALID_ARG, "timer is NULL");
    return run(plan, std::vector<void*>(bufs, bufs + plan->n),
               static_cast<hipStream_t>(stream), timer);
}

AR_EXPORT ar_status ar_plan_execute_strided(ar_plan* plan, void* base, int64_t stride_bytes,
                                            void* stream) {
    clear_error();
    if (!plan) return fail(AR_ERR_INVALID_ARG, "plan is NULL");
    if (!base) return fail(AR_ERR_INVALID_ARG, "base is NULL");
    if (stride_bytes < plan->N * plan->esize)
        return fail(AR_ERR_INVALID_ARG, "stride_bytes < N * element size");
    std::vector<void*> bufs(size_t(plan->n));
    for (int32_t i = 0; i < plan->n; ++i)
        bufs[size_t(i)] = static_cast<char*>(base) + int64_t(i) * stride_bytes;
    return run(plan, bufs, static_cast<hipStream_t>(stream), nullptr);
}

AR_EXPORT ar_status ar_timer_create(int64_t capacity, ar_timer** out) {
    clear_error();
    if (!out) return fail(AR_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (capacity < 1 || capacity > (int64_t(1) << 24))
        return fail(AR_ERR_INVALID_ARG, "capacity must be in [1, 2^24]");
    try {
        ar_timer* t = new ar_timer();
        t->cap = capacity;
        t->ev.assign(size_t(2 * capacity), nullptr);
        t->launch.assign(size_t(capacity), -1);
        *out = t;
        return AR_OK;
    } catch (const std::bad_alloc&) {
        return fail(AR_ERR_OOM, "host allocation failed");
    }
}

AR_EXPORT ar_status ar_timer_reset(ar_timer* timer) {
    clear_error();
    if (!timer) return fail(AR_ERR_INVALID_ARG, "timer is NULL");
    timer->count = 0;
    return AR_OK;
}

AR_EXPORT ar_status ar_timer_read(ar_timer* timer, int64_t cap, int64_t* count,
                                  int32_t* launch, float* ms) {
    clear_error();
    if (!timer || !count) return fail(AR_ERR_INVALID_ARG, "NULL argument");
    if (cap < 0) return fail(AR_ERR_INVALID_ARG, "cap < 0");
    const int64_t m = std::min(cap, timer->count);
    for (int64_t i = 0; i < m; ++i) {
        if (ms) {
            hipError_t e = hipEventSynchronize(timer->ev[size_t(2 * i + 1)]);
            if (e != hipSuccess) return fail(AR_ERR_HIP, hip_msg("hipEventSynchronize", e));
            float t = 0.f;
            e = hipEventElapsedTime(&t, timer->ev[size_t(2 * i)], timer->ev[size_t(2 * i + 1)]);
            if (e != hipSuccess) return fail(AR_ERR_HIP, hip_msg("hipEventElapsedTime", e));
            ms[i] = t;
        }
        if (launch) launch[i] = timer->launch[size_t(i)];
    }
    *count = m;
    return AR_OK;
}

AR_EXPORT ar_status ar_timer_destroy(ar_timer* timer) {
    clear_error();
    if (!timer) return AR_OK;
    for (hipEvent_t e : timer->ev)
        if (e) (void)hipEventDestroy(e);
    delete timer;
    return AR_OK;
}

AR_EXPORT ar_status ar_plan_set_option(ar_plan* plan, int32_t option, int64_t value) {
    clear_error();
    if (!plan) return fail(AR_ERR_INVALID_ARG, "plan is NULL");
    int32_t* field = nullptr;
    if (option == AR_OPT_FUSE) {
        if (value != 0 && value != 1) return fail(AR_ERR_INVALID_ARG, "AR_OPT_FUSE takes 0 or 1");
        field = &plan->fuse;
    } else if (option == AR_OPT_SLICE) {
        if (value < 0 || value > 2) return fail(AR_ERR_INVALID_ARG, "AR_OPT_SLICE takes 0, 1 or 2");
        field = &plan->slice;
    } else if (option == AR_OPT_RESIDENT) {
        if (value != 0 && value != 1) return fail(AR_ERR_INVALID_ARG, "AR_OPT_RESIDENT takes 0 or 1");
        field = &plan->resident;
    } else {
        return fail(AR_ERR_INVALID_ARG, "unknown option");
    }
    if (*field != int32_t(value)) {
        exec_release(*plan);
        *field = int32_t(value);
    }
    return AR_OK;
}

AR_EXPORT ar_status ar_plan_num_launches(const ar_plan* plan, int32_t* count) {
    clear_error();
    if (!plan || !count) return fail(AR_ERR_INVALID_ARG, "NULL argument");
    try {
        const ExecState* ex = exec_state(const_cast<ar_plan&>(*plan));
        *count = int32_t(ex->stages.size());
        return AR_OK;
    } catch (const std::bad_alloc&) {
        return fail(AR_ERR_OOM, "host allocation failed");
    } catch (const std::exception& e) {
        return fail(AR_ERR_INTERNAL, e.what());
    }
}

AR_EXPORT ar_status ar_plan_launch_kernel(const ar_plan* plan, int32_t i, int32_t* kernel) {
    clear_error();
    if (!plan || !kernel) return fail(AR_ERR_INVALID_ARG, "NULL argument");
    try {
        const ExecState* ex = exec_state(const_cast<ar_plan&>(*plan));
        if (i < 0 || i >= int32_t(ex->stages.size()))
            return fail(AR_ERR_INVALID_ARG, "launch index out of range");
        const Stage stg = ex->stages[size_t(i)];
        if (stg.slice >= 0) {
            const SliceDesc& sd = ex->slices[size_t(stg.slice)];
            *kernel = sd.streamed ? AR_KERNEL_STREAM : sd.resident ? AR_KERNEL_RESIDENT
                                                                   : AR_KERNEL_SLICED;
        } else if (stg.launch < 0) {
            *kernel = AR_KERNEL_ONEPASS;
        } else {
            *kernel = ex->launches[size_t(stg.launch)].dsplit > 1 ? AR_KERNEL_SPLIT
                                                                   : AR_KERNEL_PHASE;
        }
        return AR_OK;
    } catch (const std::bad_alloc&) {
        return fail(AR_ERR_OOM, "host allocation failed");
    } catch (const std::exception& e) {
        return fail(AR_ERR_INTERNAL, e.what());
    }
}

AR_EXPORT ar_status ar_plan_launch_info(const ar_plan* plan, int32_t i, int32_t* phase,
                                        int32_t* nsrc, int32_t* max_dst, int64_t* num_steps,
                                        int64_t* bytes) {
    clear_error();
    if (!plan) return fail(AR_ERR_INVALID_ARG, "plan is NULL");
    try {
        const ExecState* ex = exec_state(const_cast<ar_plan&>(*plan));
        if (i < 0 || i >= int32_t(ex->stages.size()))
            return fail(AR_ERR_INVALID_ARG, "launch index out of range");
        const Stage stg = ex->stages[size_t(i)];
        if (stg.slice >= 0) {
            const SliceDesc& sd = ex->slices[size_t(stg.slice)];
            if (phase) *phase = sd.streamed ? -3 : sd.resident ? -2 : -1;
            if (nsrc) *nsrc = sd.max_k;
            if (max_dst) *max_dst = sd.max_dst;
            if (num_steps) *num_steps = sd.nsteps;
            if (bytes) *bytes = sd.resident ? sd.res_bytes : sd.bytes;
            return AR_OK;
        }
        if (stg.launch < 0) {  // the one-pass launch
            if (phase) *phase = -4;
            if (nsrc) *nsrc = ex->one.max_k;
            if (max_dst) *max_dst = ex->one.max_dst;
            if (num_steps) *num_steps = ex->one.nsteps;
            if (bytes) *bytes = ex->one.bytes;
            return AR_OK;
        }
        const LaunchDesc& L = ex->launches[size_t(stg.launch)];
        if (phase) *phase = L.phase;
        if (nsrc) *nsrc = ex->hsteps[size_t(L.first)].k;
        if (max_dst) *max_dst = L.max_dst;
        if (num_steps) *num_steps = L.count;
        if (bytes) *bytes = L.bytes;
        return AR_OK;
    } catch (const std::bad_alloc&) {
        return fail(AR_ERR_OOM, "host allocation failed");
    } catch (const std::exception& e) {
        return fail(AR_ERR_INTERNAL, e.what());
    }
}
