// Solving every distinct instance once.
//
// A sweep over an arrival-rate trace (Section 6 drives the system with the
// per-second rates of one) hands the solver the same (rate, objective, replicas,
// profile) tuple again and again.  Equal inputs have equal answers, so only one
// instance per distinct tuple is solved:
//   k6_fill     empties the hash table;
//   k6_dedupe   one thread per instance: hash the instance's input words, find the
//               first of its workgroup with equal words in a table in LDS, and insert
//               those in the global table with open addressing (a compare and swap per
//               probe); the first index to take a slot is the representative of its
//               tuple, later ones with equal words learn it from the slot.  Writes
//               rep[i] and the list of the representatives, which are then solved;
//   k6_scatter  afterwards: every other instance copies the outputs of its
//               representative, a thread per word.
// Which index of a tuple becomes the representative depends on the order the
// threads arrive in; the outputs do not, since equal inputs have one answer.
// (Batches of up to an instance per SIMD don't come here, see themis_solve_distinct.)
//
// What bounds it: the launches (four, some four microseconds each) and, before the
// workgroups sorted out their own duplicates, the compare-and-swaps, which serialise
// per slot: of 86400 instances with 261 distinct tuples every one did one (36 us; now
// a tenth of them do, 8.6 us).  The scatter took a thread per instance, with rows of
// 72 bytes in strides (12 us, now 5.4), and the solve a wavefront per instance to find
// that it was not to be solved (25 us, now 7).  The whole call: 80 -> 21 us by the traces of
// its kernels, 24 from call to call, 20.5 with the solve as it is now.
//
// Pipelines of more than 64 models go through the three stages, which take no list:
// there the pass gets an arrival rate of zero for the instances it is not to solve,
// and "invalid" in every output, which it overwrites for those it solves.
#include "themis_internal.h"

namespace themis {
namespace {

constexpr int32_t MEMO_EMPTY = -1;

typedef int32_t memo_i32x4 __attribute__((ext_vector_type(4)));

// (the number of slots is a multiple of 256)
__global__ __launch_bounds__(256) void k6_fill(memo_i32x4* __restrict__ table, uint32_t quads,
                                               int32_t* __restrict__ count)
{
    const uint32_t g = blockIdx.x * 256u + threadIdx.x;
    if (g < quads) table[g] = memo_i32x4{MEMO_EMPTY, MEMO_EMPTY, MEMO_EMPTY, MEMO_EMPTY};
    if (g == 0u) *count = 0;
}

struct MemoIn {
    const int32_t* coef;     // [N][S][cs], or [S][cs] when shared (then not part of the tuple)
    const int32_t* lambda;   // [N]
    const int32_t* slo_us;   // [N]
    const int32_t* r_fixed;  // [N][S] or null
    int S, cs, coef_shared;
};

__device__ __forceinline__ uint32_t mix(uint32_t h, uint32_t word)
{
    h ^= word;
    h *= 0x9E3779B1u;
    return h ^ (h >> 15);
}

__device__ uint32_t hash_of(const MemoIn& in, uint32_t i)
{
    uint32_t h = mix(mix(0x243F6A88u, (uint32_t)in.lambda[i]), (uint32_t)in.slo_us[i]);
    if (in.r_fixed)
        for (int s = 0; s < in.S; ++s) h = mix(h, (uint32_t)in.r_fixed[(size_t)i * in.S + s]);
    if (!in.coef_shared) {
        const int32_t* c = in.coef + (size_t)i * in.S * in.cs;
        for (int x = 0; x < in.S * in.cs; ++x) h = mix(h, (uint32_t)c[x]);
    }
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    return h ^ (h >> 13);
}

__device__ bool same_inputs(const MemoIn& in, uint32_t a, uint32_t b)
{
    bool same = in.lambda[a] == in.lambda[b] && in.slo_us[a] == in.slo_us[b];
    if (same && in.r_fixed)
        for (int s = 0; s < in.S; ++s)
            same = same && in.r_fixed[(size_t)a * in.S + s] == in.r_fixed[(size_t)b * in.S + s];
    if (same && !in.coef_shared) {
        const int32_t* ca = in.coef + (size_t)a * in.S * in.cs;
        const int32_t* cb = in.coef + (size_t)b * in.S * in.cs;
        for (int x = 0; x < in.S * in.cs; ++x) same = same && ca[x] == cb[x];
    }
    return same;
}

struct MemoOut {
    int32_t *status, *cost, *ticks, *cfg;
};

constexpr uint32_t MEMO_THREADS = 1024, MEMO_LOCAL = 2048;

// LIST: representatives are listed in `pass`; else `pass` takes their arrival rates
// (zero for the others) and the outputs "invalid".
template <bool LIST>
__global__ __launch_bounds__(MEMO_THREADS) void k6_dedupe(
    MemoIn in, int32_t* __restrict__ table, uint32_t slots, int32_t* __restrict__ rep,
    int32_t* __restrict__ pass, int32_t* __restrict__ count, int32_t* __restrict__ tmeta,
    MemoOut out, uint32_t N)
{
    __shared__ int32_t local[MEMO_LOCAL];    // thread that stands for a tuple, by hash
    __shared__ uint32_t hashes[MEMO_THREADS];
    __shared__ int32_t reps[MEMO_THREADS];
    __shared__ int32_t listed, list_at;
    const uint32_t tid = threadIdx.x;
    for (uint32_t x = tid; x < MEMO_LOCAL; x += MEMO_THREADS) local[x] = MEMO_EMPTY;
    if (tid == 0u) listed = 0;
    const uint32_t i = blockIdx.x * MEMO_THREADS + tid;
    const uint32_t first = blockIdx.x * MEMO_THREADS;
    const bool there = i < N;
    const uint32_t h = there ? hash_of(in, i) : 0u;
    hashes[tid] = h;
    __syncthreads();
    // Twice as many slots as threads in LDS, and at least twice as many as instances in
    // the global table: a probe sequence meets an empty slot (or an equal instance)
    // long before it has gone round; the bounds make the loops finite whatever the
    // tables hold.
    uint32_t who = tid;
    if (there) {
        for (uint32_t probe = 0; probe < MEMO_LOCAL; ++probe) {
            const int32_t seen = atomicCAS(&local[(h + probe) & (MEMO_LOCAL - 1u)], MEMO_EMPTY,
                                           (int32_t)tid);
            if (seen == MEMO_EMPTY) break;
            if (hashes[seen] == h && same_inputs(in, i, first + (uint32_t)seen)) {
                who = (uint32_t)seen;
                break;
            }
        }
        if (who == tid) {
            int32_t mine = (int32_t)i;
            for (uint32_t probe = 0; probe < slots; ++probe) {
                int32_t* const slot = &table[(h + probe) & (slots - 1u)];
                // (a stale "empty" is put right by the swap)
                int32_t seen = *(volatile int32_t*)slot;
                if (seen == MEMO_EMPTY) seen = atomicCAS(slot, MEMO_EMPTY, (int32_t)i);
                if (seen == MEMO_EMPTY) break;
                if ((uint32_t)seen < N && same_inputs(in, i, (uint32_t)seen)) {
                    mine = seen;
                    break;
                }
            }
            reps[tid] = mine;
        }
    }
    __syncthreads();
    const int32_t mine = there ? reps[who] : 0;
    const bool stands = there && mine == (int32_t)i;
    if (LIST) {
        // one reservation per workgroup
        int32_t at = 0;
        if (stands) at = atomicAdd(&listed, 1);
        __syncthreads();
        if (tid == 0u) list_at = listed ? atomicAdd(count, listed) : 0;
        __syncthreads();
        if (stands) pass[list_at + at] = (int32_t)i;
        // an instance that is not solved has no tables to look at
        if (there) tmeta[i] = -1;
    }
    if (!there) return;
    rep[i] = mine;
    if (!LIST) {
        pass[i] = stands ? in.lambda[i] : 0;
        out.status[i] = THEMIS_INVALID;
        out.cost[i] = -1;
        out.ticks[i] = -1;
        for (int x = 0; x < 3 * in.S; ++x) out.cfg[(size_t)i * 3 * in.S + x] = 0;
    }
}

// thread g: word g of the configurations; the first N threads the other outputs as well.
// width = 3 S; magic = ceil(2^32 / width), exact while N * width^2 < 2^32, else 0.
__global__ __launch_bounds__(256) void k6_scatter(const int32_t* __restrict__ rep, MemoOut out,
                                                  uint32_t N, uint32_t words, uint32_t width,
                                                  uint32_t magic)
{
    const uint32_t g = blockIdx.x * 256u + threadIdx.x;
    if (g >= words) return;
    const uint32_t i = magic ? __umulhi(g, magic) : g / width;
    const uint32_t r = (uint32_t)rep[i];
    // representatives are never written here, so reading theirs races with nothing
    if (r != i && r < N) out.cfg[g] = out.cfg[(size_t)r * width + (g - i * width)];
    if (g < N) {
        const uint32_t rg = (uint32_t)rep[g];
        if (rg != g && rg < N) {
            out.status[g] = out.status[rg];
            out.cost[g] = out.cost[rg];
            out.ticks[g] = out.ticks[rg];
        }
    }
}

}  // namespace

hipError_t launch_memo_dedupe(const themis_problem_t& p, const Layout& L, const MemoLayout& M,
                              const int32_t* d_coef, const int32_t* d_lambda,
                              const int32_t* d_slo_us, const int32_t* d_r_fixed,
                              int32_t* d_status, int32_t* d_cost, int32_t* d_ticks,
                              int32_t* d_cfg, char* ws, hipStream_t st)
{
    int32_t* const table = (int32_t*)(ws + M.table_off);
    int32_t* const count = (int32_t*)(ws + L.ctrl_off) + LIST_WORD;
    const uint32_t quads = M.slots / 4u;
    hipLaunchKernelGGL(k6_fill, dim3((quads + 255u) / 256u), dim3(256), 0, st, (memo_i32x4*)table,
                       quads, count);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    MemoIn in{};
    in.coef = d_coef;
    in.lambda = d_lambda;
    in.slo_us = d_slo_us;
    in.r_fixed = d_r_fixed;
    in.S = L.S;
    in.cs = p.profile_form == THEMIS_PROFILE_EQ1 ? 6 : 5;
    in.coef_shared = p.coef_shared;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(((uint32_t)L.N + MEMO_THREADS - 1u) / MEMO_THREADS),
                           dim3(MEMO_THREADS), 0, st, in, table, M.slots,
                           (int32_t*)(ws + M.rep_off), (int32_t*)(ws + M.pass_off), count,
                           (int32_t*)(ws + L.tmeta_off), MemoOut{d_status, d_cost, d_ticks, d_cfg},
                           (uint32_t)L.N);
        return hipGetLastError();
    };
    return cost_solve_serves(L) ? launch(&k6_dedupe<true>) : launch(&k6_dedupe<false>);
}

hipError_t launch_memo_scatter(const Layout& L, const MemoLayout& M, int32_t* d_status,
                               int32_t* d_cost, int32_t* d_ticks, int32_t* d_cfg, const char* ws,
                               hipStream_t st)
{
    // N S < 2^28 and S <= 32767, so the words fit 32 bits and i * width does
    const uint32_t width = 3u * (uint32_t)L.S, words = (uint32_t)L.N * width;
    const uint32_t magic = (uint64_t)words * width < (1ull << 32)
                               ? (uint32_t)(((1ull << 32) + width - 1u) / width)
                               : 0u;
    hipLaunchKernelGGL(k6_scatter, dim3((words + 255u) / 256u), dim3(256), 0, st,
                       (const int32_t*)(ws + M.rep_off), MemoOut{d_status, d_cost, d_ticks, d_cfg},
                       (uint32_t)L.N, words, width, magic);
    return hipGetLastError();
}

}  // namespace themis
