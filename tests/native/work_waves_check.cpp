// host-only check of build_work_waves over random layouts: every sub-block of every tile belongs to
// exactly one wavefront of the launch that carries its parameter group, runs name the wavefronts of
// one parameter tile, or of one chunk's RAW tiles, that share a workgroup, launches begin at workgroups
#include "layout.hpp"
#include <cstdio>
#include <random>
using namespace ffsnap;
int main(){
  std::mt19937_64 rng(2);
  static char arena[1<<16];
  for(int it=0; it<2000; it++){
    std::vector<ff_segment> segs;
    const uint64_t chunk = 1024ull << (rng()%14);
    const uint32_t per_launch = 1 + rng()%5;
    const int np = 1 + rng()%12;
    for(int p=0;p<np;p++){
      const uint64_t ne = rng()%3==0 ? 1 + rng()%5 : 1 + rng()%40000;
      segs.push_back({arena+2, 2*ne, FF_BF16, FF_KIND_W16, (uint32_t)p, 0});
      for(uint32_t k=FF_KIND_MASTER;k<=FF_KIND_V;k++) segs.push_back({arena+4, 4*ne, FF_F32, k, (uint32_t)p, 0});
      if(rng()%3==0) segs.push_back({arena+2, 2*(rng()%60000), FF_BF16, FF_KIND_RAW, 0, 0});
      for(uint64_t k=rng()%30; k-- && rng()%8;) segs.push_back({arena+2, 2*(1+rng()%3000), FF_BF16, FF_KIND_RAW, 0, 0});
    }
    Layout L;
    if(build_layout(segs.data(), segs.size(), chunk, 0, L)!=FF_OK) continue;
    std::vector<WorkTile> tiles; build_work_tiles(L,tiles);
    std::vector<WorkWave> w; std::vector<uint32_t> begin;
    if(!build_work_waves(tiles, L.params.size(), per_launch, w, begin)){ printf("refused\n"); return 1; }
    { // the limit is on the entries themselves, whatever their number for each tile
      std::vector<WorkWave> w2; std::vector<uint32_t> begin2;
      if(!build_work_waves(tiles, L.params.size(), per_launch, w2, begin2, w.size()) || begin2!=begin ||
         build_work_waves(tiles, L.params.size(), per_launch, w2, begin2, w.size()-1)){ printf("limit\n"); return 1; }
    }
    const uint64_t launches = (L.params.size()+per_launch-1)/per_launch;
    if(begin.size()!=launches+1 || begin[0]!=0 || begin.back()!=w.size()){ printf("launches\n"); return 1; }
    std::vector<uint32_t> seen(tiles.size(), 0);
    for(uint64_t k=0;k<launches;k++){
      if(begin[k]%kWavesPerGroup || begin[k]>begin[k+1]){ printf("launch begin\n"); return 1; }
      for(uint32_t i=begin[k];i<begin[k+1];i++){
        if(w[i].tile==kNoTile) continue;
        const WorkTile& t=tiles[w[i].tile];
        if(t.kind==kWorkParam ? t.grad_index/per_launch!=k : k+1!=launches){ printf("launch of a tile\n"); return 1; }
        const uint32_t sub=w[i].info&15, first=(w[i].info>>4)&7, len=(w[i].info>>8)&15;
        if(seen[w[i].tile]&(1u<<sub)){ printf("twice\n"); return 1; }
        seen[w[i].tile]|=1u<<sub;
        const uint32_t slot=i%kWavesPerGroup, base=i-slot;
        if(slot<first || slot>=first+len || first+len>kWavesPerGroup){ printf("run place\n"); return 1; }
        for(uint32_t s=0;s<kWavesPerGroup;s++){
          const bool in = s>=first && s<first+len;
          const uint32_t o=w[base+s].tile;
          // RAW tiles of one chunk share a run, they are neighbours in the stream
          const bool mates = o==w[i].tile || (o!=kNoTile && t.kind==kWorkRaw && tiles[o].kind==kWorkRaw && tiles[o].chunk[0]==t.chunk[0]);
          if(in != mates){ printf("run members\n"); return 1; }
          if(in && ((w[base+s].info>>4)!=(w[i].info>>4))){ printf("run of a mate\n"); return 1; }
        }
      }
    }
    for(size_t i=0;i<tiles.size();i++){
      const WorkTile& t=tiles[i];
      const bool par=t.kind==kWorkParam;
      const uint64_t a = par ? t.e0%kParamTileElems : t.soff[0]%kRawTileBytes, size = par ? kSubElems : kSubRawBytes;
      if(t.n==0 || a+t.n > (par?kParamTileElems:kRawTileBytes)){ printf("block\n"); return 1; }
      uint32_t want=0;
      for(uint64_t s=a/size; s<=(a+t.n-1)/size; s++) want|=1u<<s;
      if(seen[i]!=want){ printf("cover %zu\n",i); return 1; }
    }
  }
  printf("ok\n"); return 0;
}
