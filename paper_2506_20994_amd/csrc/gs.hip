// Gather-scatter sum u <- Q Q^T u (paper Sec. 2.1).
//
// Plan: only ids that occur more than once need work.  Those "shared" ids are
// listed in the order their first local copy appears (so neighbouring threads
// touch neighbouring memory), each with its local copies (sem::Copies).  One
// thread per shared id sums its copies in increasing local index and writes the
// sum back to every copy: deterministic, no atomics.
//
// Negative ids mark Dirichlet nodes (homogeneous Dirichlet conditions): they
// are no unknowns.  They take no unique index (lid = -1), sit after every
// unique node's copies in the CSR order (positions n_local - n_masked ..
// n_local of uidx, in increasing local index), and gather-scatter sets them to
// zero.  Their multiplicity is 1 and their owner weight 0.
#include <algorithm>
#include <vector>

#include "sem_internal.h"

namespace {

constexpr int kBlock = 256;

// Bound by the lines of the local layout (an element's faces touch every line of it:
// 325 MB at 32^3, lx 8, for 211 MB of values and indices) and the chain link, more,
// values: with both of a node's entries of more read at once and kept for the stores
// 85.5 us there and 12.6 us at 19^3, lx 7 (one entry at a time, read again for the
// stores: 88.5 and 13.7; three index lists per node: 87.0 and 12.6; 256 and 1024
// threads a workgroup: 86.4 and 87.8).
// threads [0, n_shared) sum the shared ids; threads [n_shared, n_shared +
// n_masked) zero the Dirichlet nodes listed in midx
template <typename T>
__global__ void gs_kernel(T* __restrict__ u, sem::Copies cp, int64_t n_shared, const int* __restrict__ skip,
                          const int32_t* __restrict__ midx, int64_t n_masked) {
    if (skip && *skip) return;
    const int64_t g = sem::xcd_order(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (g >= n_shared) {
        if (g < n_shared + n_masked) u[midx[g - n_shared]] = T(0);
        return;
    }
    const sem::NodeCopies n = sem::node_copies(cp, g);
    const T s = sem::sum_copies_flat<T>(cp, n, [=](int32_t L) { return u[L]; });
    u[n.c.x] = s;
    if (n.c.y >= 0) u[n.c.y] = s;
    if (n.i.x >= 0) {
        u[n.i.x] = s;
        u[n.i.y] = s;
    }
    if (n.i.z >= 0) u[n.i.z] = s;
    if (n.j.x >= 0) u[n.j.x] = s;
    if (n.j.y >= 0) u[n.j.y] = s;
    if (n.j.z >= 0) u[n.j.z] = s;
    if (n.j.w >= 0) u[n.j.w] = s;
    for (int k = 2; k <= n.i.w; ++k) {
        const int4 j = cp.more[-2 - n.c.y + k];
        u[j.x] = s;
        if (j.y >= 0) u[j.y] = s;
        if (j.z >= 0) u[j.z] = s;
        if (j.w >= 0) u[j.w] = s;
    }
}

// int4 entries that a node of m copies takes in sem::Copies::more
__host__ __device__ inline int64_t more_entries(int32_t m) { return m < 3 ? 0 : 1 + (m > 4 ? (m - 1) / 4 : 0); }

// link[u] and more from the CSR lists; *next counts the entries of more handed
// out, a workgroup's at a time (their order differs from build to build, what
// they hold does not)
__global__ void link_kernel(int2* __restrict__ link, int4* __restrict__ more, unsigned* __restrict__ next,
                            const int32_t* __restrict__ uoff, const int32_t* __restrict__ uidx, int64_t nu) {
    __shared__ unsigned s_count, s_base;
    for (int64_t u0 = blockIdx.x * (int64_t)blockDim.x; u0 < nu; u0 += (int64_t)gridDim.x * blockDim.x) {
        const int64_t u = u0 + threadIdx.x;
        const int32_t b = u < nu ? uoff[u] : 0, m = u < nu ? uoff[u + 1] - b : 1;
        const unsigned n = (unsigned)more_entries(m);
        if (threadIdx.x == 0) s_count = 0;
        __syncthreads();
        const unsigned mine = n ? atomicAdd(&s_count, n) : 0;
        __syncthreads();
        if (threadIdx.x == 0 && s_count) s_base = atomicAdd(next, s_count);
        __syncthreads();
        if (u < nu) {
            int2 c{uidx[b], m == 2 ? uidx[b + 1] : -1};
            if (n) {
                const int32_t q = (int32_t)(s_base + mine);
                c.y = -2 - q;
                auto at = [&](int32_t k) { return k < m ? uidx[b + k] : -1; };
                more[q] = int4{at(1), at(2), at(3), (int32_t)n - 1};
                for (int32_t k = 1; k < (int32_t)n; ++k)
                    more[q + k] = int4{at(4 * k), at(4 * k + 1), at(4 * k + 2), at(4 * k + 3)};
            }
            link[u] = c;
        }
        __syncthreads();
    }
}

// slink[g] = link of the g-th shared id, unique node su[g]
__global__ void slink_kernel(int2* __restrict__ slink, const int2* __restrict__ link, const int32_t* __restrict__ su,
                             int64_t n_shared) {
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g < n_shared) slink[g] = link[su[g]];
}

// multiplicity and owner weight of every local node: threads [0, nu) the copies of a
// unique node (ascending: the first owns), threads [nu, nu + n_masked) a Dirichlet node
__global__ void weights_kernel(double* __restrict__ mult, double* __restrict__ owner, const int32_t* __restrict__ uoff,
                               const int32_t* __restrict__ uidx, int64_t nu, int64_t n_masked) {
    const int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (u < nu) {
        const int32_t b = uoff[u], e = uoff[u + 1];
        for (int32_t q = b; q < e; ++q) {
            const int32_t L = uidx[q];
            mult[L] = (double)(e - b);
            owner[L] = q == b ? 1.0 : 0.0;
        }
    } else if (u < nu + n_masked) {
        const int32_t L = uidx[uoff[nu] + (u - nu)];
        mult[L] = 1.0;
        owner[L] = 0.0;
    }
}

}  // namespace

extern "C" int sem_gs_setup(sem_ctx_t ctx, const int64_t* ids, int64_t n_local, sem_gs_t* out) {
    int rc = sem::enter(ctx);
    if (rc) return rc;
    if (!out) return sem::fail(ctx, SEM_EINVAL, "sem_gs_setup: null output pointer");
    *out = nullptr;
    if (n_local < 0 || n_local >= ((int64_t)1 << 31))
        return sem::fail(ctx, SEM_EINVAL, "sem_gs_setup: n_local=%lld outside [0, 2^31)", (long long)n_local);
    if (n_local > 0 && !ids) return sem::fail(ctx, SEM_EINVAL, "sem_gs_setup: null ids");
    int64_t idmax = -1, n_masked = 0;
    for (int64_t L = 0; L < n_local; ++L) {
        if (ids[L] < 0) ++n_masked;
        else idmax = std::max(idmax, ids[L]);
    }
    // Dense relabelling when ids are sparse: map them onto 0..n_distinct-1 by
    // their sorted order, so the counting arrays stay O(n_local).
    std::vector<int64_t> relabel;
    const int64_t* key = ids;
    if (idmax > 4 * n_local + 1024) {
        std::vector<int64_t> uniq;
        uniq.reserve((size_t)(n_local - n_masked));
        for (int64_t L = 0; L < n_local; ++L)
            if (ids[L] >= 0) uniq.push_back(ids[L]);
        std::sort(uniq.begin(), uniq.end());
        uniq.erase(std::unique(uniq.begin(), uniq.end()), uniq.end());
        relabel.resize((size_t)n_local);
        for (int64_t L = 0; L < n_local; ++L)
            relabel[(size_t)L] = ids[L] < 0 ? -1 : std::lower_bound(uniq.begin(), uniq.end(), ids[L]) - uniq.begin();
        idmax = (int64_t)uniq.size() - 1;
        key = relabel.data();
    }
    // count copies per id
    std::vector<int32_t> count((size_t)(idmax + 1), 0);
    for (int64_t L = 0; L < n_local; ++L)
        if (key[L] >= 0) ++count[(size_t)key[L]];
    int64_t n_unique = 0;
    int64_t n_more = 0;
    for (int32_t c : count) {
        n_unique += (c > 0);
        n_more += more_entries(c);
    }
    // dense unique numbering in order of first appearance and the CSR of the
    // local copies of every unique node, slot[id] = unique index or -1; the shared ids
    // are the unique nodes of several copies, listed behind the counter of link_kernel
    std::vector<int32_t> slot((size_t)(idmax + 1), -1);
    std::vector<int32_t> shared(1, 0);
    std::vector<int32_t> lid((size_t)n_local);
    std::vector<int32_t> uoff(1, 0);
    uoff.reserve((size_t)n_unique + 1);
    int32_t nu = 0;
    for (int64_t L = 0; L < n_local; ++L) {
        const int64_t g = key[L];
        if (g < 0) {
            lid[(size_t)L] = -1;
            continue;
        }
        if (slot[(size_t)g] < 0) {
            if (count[(size_t)g] > 1) shared.push_back(nu);
            slot[(size_t)g] = nu++;
            uoff.push_back(uoff.back() + count[(size_t)g]);
        }
        lid[(size_t)L] = slot[(size_t)g];
    }
    // CSR positions: the copies of every unique node, then the Dirichlet nodes
    std::vector<int32_t> uidx((size_t)n_local), upos((size_t)n_local);
    {
        std::vector<int32_t> pos(uoff.begin(), uoff.end() - 1);
        int32_t tail = uoff.back();
        for (int64_t L = 0; L < n_local; ++L) {
            const int32_t u = lid[(size_t)L];
            const int32_t q = u >= 0 ? pos[(size_t)u]++ : tail++;
            uidx[(size_t)q] = (int32_t)L;
            upos[(size_t)L] = q;
        }
    }
    std::vector<int32_t>().swap(count);
    std::vector<int32_t>().swap(slot);

    const int64_t n_shared = (int64_t)shared.size() - 1;
    auto* gs = new sem_gs_s();
    gs->ctx = ctx;
    gs->n_local = n_local;
    gs->n_unique = n_unique;
    gs->n_shared = n_shared;
    gs->n_masked = n_masked;
    hipError_t e = hipSuccess;
    auto alloc = [&](auto** p, size_t bytes) {
        if (e == hipSuccess && bytes) e = hipMalloc(p, bytes);
    };
    auto upload = [&](int32_t* p, const std::vector<int32_t>& v) {
        if (e == hipSuccess && !v.empty())
            e = hipMemcpy(p, v.data(), sizeof(int32_t) * v.size(), hipMemcpyHostToDevice);
    };
    if (n_unique > 0) alloc(&gs->more, sizeof(int4) * n_more + sizeof(int2) * (n_unique + n_shared));
    if (e == hipSuccess && n_unique > 0) {
        gs->link = reinterpret_cast<int2*>(gs->more + n_more);
        gs->slink = gs->link + n_unique;
    }
    alloc(&gs->mult, sizeof(double) * n_local);
    alloc(&gs->owner, sizeof(double) * n_local);
    alloc(&gs->lid, sizeof(int32_t) * n_local);
    alloc(&gs->uidx, sizeof(int32_t) * n_local);
    alloc(&gs->upos, sizeof(int32_t) * n_local);
    alloc(&gs->uoff, sizeof(int32_t) * uoff.size());
    upload(gs->upos, upos);
    upload(gs->lid, lid);
    upload(gs->uidx, uidx);
    upload(gs->uoff, uoff);
    // the shared ids and their counter lie where the multiplicities go once the links
    // are made (at most n_local / 2 of them): no memory of their own to free
    int32_t* d_shared = reinterpret_cast<int32_t*>(gs->mult);
    if (n_unique > 0) upload(d_shared, shared);
    if (e == hipSuccess && n_local > 0) {
        hipStream_t st = ctx->stream;
        auto blocks = [](int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); };
        if (n_unique > 0) {
            link_kernel<<<std::min(blocks(n_unique), 4096u), kBlock, 0, st>>>(
                gs->link, gs->more, reinterpret_cast<unsigned*>(d_shared), gs->uoff, gs->uidx, n_unique);
            e = hipGetLastError();
        }
        if (e == hipSuccess && n_shared > 0) {
            slink_kernel<<<blocks(n_shared), kBlock, 0, st>>>(gs->slink, gs->link, d_shared + 1, n_shared);
            e = hipGetLastError();
        }
        if (e == hipSuccess) {
            weights_kernel<<<blocks(n_unique + n_masked), kBlock, 0, st>>>(gs->mult, gs->owner, gs->uoff, gs->uidx,
                                                                           n_unique, n_masked);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipStreamSynchronize(st);
    }
    if (e != hipSuccess) {
        sem_gs_destroy(gs);
        return sem::check_hip(ctx, e, "sem_gs_setup");
    }
    *out = gs;
    return SEM_OK;
}

extern "C" int sem_gs_destroy(sem_gs_t gs) {
    if (!gs) return SEM_OK;
    if (gs->ctx) (void)hipSetDevice(gs->ctx->device);
    if (gs->more) (void)hipFree(gs->more);
    if (gs->mult) (void)hipFree(gs->mult);
    if (gs->owner) (void)hipFree(gs->owner);
    if (gs->lid) (void)hipFree(gs->lid);
    if (gs->uoff) (void)hipFree(gs->uoff);
    if (gs->uidx) (void)hipFree(gs->uidx);
    if (gs->upos) (void)hipFree(gs->upos);
    delete gs;
    return SEM_OK;
}

extern "C" int sem_gs_info(sem_gs_t gs, int64_t* n_unique, int64_t* n_shared) {
    if (!gs) return sem::fail(nullptr, SEM_EINVAL, "sem_gs_info: null plan");
    if (n_unique) *n_unique = gs->n_unique;
    if (n_shared) *n_shared = gs->n_shared;
    return SEM_OK;
}

extern "C" int sem_gs_dirichlet_count(sem_gs_t gs, int64_t* n_dirichlet) {
    if (!gs) return sem::fail(nullptr, SEM_EINVAL, "sem_gs_dirichlet_count: null plan");
    if (n_dirichlet) *n_dirichlet = gs->n_masked;
    return SEM_OK;
}

namespace sem {

int gs_launch(sem_gs_t gs, void* u, sem_dtype_t dtype, const int* skip) {
    sem_ctx_t ctx = gs->ctx;
    const int64_t nt = gs->n_shared + gs->n_masked;
    if (nt == 0) return SEM_OK;
    if (!u) return fail(ctx, SEM_EINVAL, "sem_gs: null field");
    constexpr int kGsBlock = 512;
    const unsigned grid = (unsigned)((nt + 8 * kGsBlock - 1) / (8 * kGsBlock) * 8);   // a multiple of 8
    const int32_t* midx = gs->uidx + (gs->n_local - gs->n_masked);
    const Copies cp{gs->slink, gs->more};
    if (dtype == SEM_F64)
        gs_kernel<double><<<grid, kGsBlock, 0, ctx->stream>>>((double*)u, cp, gs->n_shared, skip,
                                                              midx, gs->n_masked);
    else if (dtype == SEM_F32)
        gs_kernel<float><<<grid, kGsBlock, 0, ctx->stream>>>((float*)u, cp, gs->n_shared, skip,
                                                             midx, gs->n_masked);
    else
        return fail(ctx, SEM_EINVAL, "sem_gs: dtype %d not supported (F64 or F32)", (int)dtype);
    SEM_LAUNCH_CHECK(ctx);
    return SEM_OK;
}

}  // namespace sem

extern "C" int sem_gs(sem_gs_t gs, void* u, sem_dtype_t dtype) {
    if (!gs) return sem::fail(nullptr, SEM_EINVAL, "sem_gs: null plan");
    int rc = sem::enter(gs->ctx);
    if (rc) return rc;
    return sem::gs_launch(gs, u, dtype, nullptr);
}

extern "C" int sem_gs_mult(sem_gs_t gs, double* mult) {
    if (!gs) return sem::fail(nullptr, SEM_EINVAL, "sem_gs_mult: null plan");
    sem_ctx_t ctx = gs->ctx;
    int rc = sem::enter(ctx);
    if (rc) return rc;
    if (gs->n_local == 0) return SEM_OK;
    if (!mult) return sem::fail(ctx, SEM_EINVAL, "sem_gs_mult: null output");
    SEM_HIP(ctx, hipMemcpyAsync(mult, gs->mult, sizeof(double) * gs->n_local,
                                hipMemcpyDeviceToDevice, ctx->stream));
    return SEM_OK;
}

extern "C" int sem_gs_owner(sem_gs_t gs, double* wgt) {
    if (!gs) return sem::fail(nullptr, SEM_EINVAL, "sem_gs_owner: null plan");
    sem_ctx_t ctx = gs->ctx;
    int rc = sem::enter(ctx);
    if (rc) return rc;
    if (gs->n_local == 0) return SEM_OK;
    if (!wgt) return sem::fail(ctx, SEM_EINVAL, "sem_gs_owner: null output");
    SEM_HIP(ctx, hipMemcpyAsync(wgt, gs->owner, sizeof(double) * gs->n_local,
                                hipMemcpyDeviceToDevice, ctx->stream));
    return SEM_OK;
}
